"""The FP64 evaluation and parameter gradient where the last workgroup of 16 centers is
partly filled, one and two species: energies, forces and virial within 1e-12 (sums of about a
hundred FP64 terms of order one: 100 x 2^-53 with two orders to spare), gradients within the
bar of the FP64 gradient, 1e-11 |ref| + 1e-13 max|ref| per block."""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_atoms", [1, 15, 17, 251])
@pytest.mark.parametrize("species", [1, 2])
def test_partly_filled_workgroups(n_atoms, species):
    say(f"case: FP64, {n_atoms} atoms, {species} species")
    hp = I.HParams(n_types=species)
    params = I.random_model(hp, 20 + species)
    at = I.fcc_box(4, 0.1, 31)
    rng = np.random.default_rng(32)
    keep = np.sort(rng.choice(at.n, n_atoms, replace=False))
    at = I.Atoms(x=np.ascontiguousarray(at.x[keep]), types=rng.integers(0, species, n_atoms).astype(np.int32),
                 box=at.box, masses=np.full(species, I.CU_MASS_AMU))
    s = make_system(at, hp, params)
    E, W, F, U = s.compute(precision="fp64", per_atom=True)
    m = oracle.Model.from_hparams(hp, params)
    Eo, Wo, Uo, Fo = oracle.evaluate(m, at.x, at.types, at.box)
    for a, b in ((U, Uo), (F, Fo), (W / n_atoms, Wo / n_atoms)):
        assert np.abs(a - b).max() < 1e-12
    assert abs(E - Eo) / n_atoms < 1e-12
    gF = rng.normal(size=(n_atoms, 3))
    for weights in (gF, None):
        g = s.train_backward64(0.7, weights).cpu().numpy()
        ref = oracle.param_grad(m, at.x, at.types, at.box, 0.7, weights)
        for a, b in hp.offsets().values():
            bar = 1e-11 * np.abs(ref[a:b]) + 1e-13 * np.abs(ref[a:b]).max()
            assert (np.abs(g[a:b] - ref[a:b]) <= bar).all()
