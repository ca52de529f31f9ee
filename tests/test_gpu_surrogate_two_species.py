"""The l <= 2 shape with two species at each lane count of evaluation and of training gradient,
against the FP64 oracle: bars of the FP32 path (per-atom energy 1e-6 eV, forces 1e-4 eV/A, virial
1e-6 eV per atom and component; gradients 1e-4 |ref| + 1e-5 max|ref| of their block), and of the
deterministic form against the default one (forces 1e-6 eV/A, energy and virial equal)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd.nep import network_params
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


def _box(n_atoms, seed):
    cells = 4
    while 4 * cells ** 3 < n_atoms:
        cells += 1
    at = I.fcc_box(cells, 0.08, seed)
    rng = np.random.default_rng(seed + 1)
    keep = np.sort(rng.choice(at.n, size=n_atoms, replace=False))
    return I.Atoms(x=np.ascontiguousarray(at.x[keep]), types=rng.integers(0, 2, n_atoms).astype(np.int32), box=at.box,
                   masses=np.array([60.0, 90.0]))


@pytest.mark.parametrize("n_atoms", [300, 8192, 8193, 16385, 32769])   # 16, 16, 8, 4, 2 lanes
def test_evaluation(n_atoms):
    say(f"case: l <= 2 shape, two species, {n_atoms} atoms, as surrogate of a full model")
    hp = I.HParams(n_types=2)
    shp = dataclasses.replace(I.SURROGATE_SHORTER_HPARAMS, n_types=2, zbl_z=(29.0, 29.0))
    params = I.random_model(hp, 3)
    sp = I.surrogate_from_teacher(hp, params, shp, 4)
    at = _box(n_atoms, 50)
    s = make_system(at, hp, params, shp, sp)
    E, W, F, U = s.compute(slot=1, per_atom=True)
    s.set_deterministic(True)
    Ed, Wd, Fd, Ud = s.compute(slot=1, per_atom=True)
    Eo, Wo, Uo, Fo = oracle.evaluate(oracle.Model.from_hparams(shp, sp), at.x, at.types, at.box)
    assert np.abs(U - Uo).max() < 1e-6 and abs(E - Eo) / at.n < 1e-6
    assert np.abs(F - Fo).max() < 1e-4 and np.abs(W - Wo).max() / at.n < 1e-6
    assert Ed == E and np.array_equal(Wd, W) and np.array_equal(Ud, U) and np.abs(Fd - F).max() < 1e-6


@pytest.mark.parametrize("n_atoms", [3, 250, 4096, 4097])   # 16 lanes, 4 lanes
def test_gradients(n_atoms):
    say(f"case: l <= 2 shape, two species, {n_atoms} atoms, gradients of network and coefficients")
    hp = dataclasses.replace(I.SURROGATE_HPARAMS, n_types=2, zbl_z=(29.0, 29.0))
    params = I.random_model(hp, 13)
    at = _box(n_atoms, 21)
    s = make_system(at, hp, params)
    rng = np.random.default_rng(4)
    gE, gF = 0.6, rng.normal(size=(at.n, 3))
    gFt = torch.tensor(gF, dtype=torch.float32, device="cuda")
    ref = oracle.param_grad(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box, gE, gF)
    p32 = torch.tensor(params, dtype=torch.float32, device="cuda")
    s.train_forward_params(0, p32)
    g = s.train_backward_params(0, p32, gE, gFt).cpu().numpy()
    th = torch.tensor(network_params(hp, params), dtype=torch.float32, device="cuda")
    gn = s.train_backward(0, th, gE, gFt).cpu().numpy()
    off = hp.offsets()
    net = off["W0"][0]
    for k in [slice(*off[b]) for b in ("cR", "cA", "sigma")] + [slice(net, None)]:
        assert (np.abs(g[k] - ref[k]) <= 1e-4 * np.abs(ref[k]) + 1e-5 * np.abs(ref[k]).max()).all()
    assert (np.abs(gn - ref[net:]) <= 1e-4 * np.abs(ref[net:]) + 1e-5 * np.abs(ref[net:]).max()).all()
