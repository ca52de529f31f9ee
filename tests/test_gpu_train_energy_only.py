"""Training gradients of an energy term alone (no force weights), whose kernel leaves the JVP out,
against the oracle's FP64 gradient at each lane count: |g - ref| <= 1e-4 |ref| + 1e-5 max|ref| of
the block, the bar of the training gradients; and against the gradient with force weights of zero,
which sums the same terms and zeros."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd.nep import network_params
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_atoms", [3, 4096, 4097, 16385])
@pytest.mark.parametrize("shape,species", [("full", 1), ("full", 2), ("surrogate", 1), ("surrogate", 2)])
def test_energy_gradient(n_atoms, shape, species):
    say(f"case: {shape} shape, {species} species, {n_atoms} atoms, energy term only")
    base = I.FULL_HPARAMS if shape == "full" else I.SURROGATE_HPARAMS
    hp = I.HParams(n_types=species, l_max_3b=base.l_max_3b, l_max_4b=base.l_max_4b, n_hidden=base.n_hidden)
    params = I.random_model(hp, 11 + species)
    cells = 4
    while 4 * cells ** 3 < n_atoms:
        cells += 1
    at = I.fcc_box(cells, 0.1, 21)
    rng = np.random.default_rng(22)
    keep = np.sort(rng.choice(at.n, size=n_atoms, replace=False))
    at = I.Atoms(x=np.ascontiguousarray(at.x[keep]), types=rng.integers(0, species, n_atoms).astype(np.int32), box=at.box,
                 masses=np.full(species, I.CU_MASS_AMU))
    s = make_system(at, hp, params)
    ref = oracle.param_grad(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box, 0.6, None)
    p32 = torch.tensor(params, dtype=torch.float32, device="cuda")
    th = torch.tensor(network_params(hp, params), dtype=torch.float32, device="cuda")
    zero = torch.zeros((at.n, 3), dtype=torch.float32, device="cuda")
    s.train_forward_params(0, p32)
    g, gz = (s.train_backward_params(0, p32, 0.6, w).cpu().numpy() for w in (None, zero))
    gn, gnz = (s.train_backward(0, th, 0.6, w).cpu().numpy() for w in (None, zero))
    off = hp.offsets()
    net = off["W0"][0]
    for k in [slice(*off[b]) for b in ("cR", "cA", "sigma")] + [slice(net, None)]:
        bar = 1e-4 * np.abs(ref[k]) + 1e-5 * np.abs(ref[k]).max()
        assert (np.abs(g[k] - ref[k]) <= bar).all() and (np.abs(gz[k] - ref[k]) <= bar).all()
    bar = 1e-4 * np.abs(ref[net:]) + 1e-5 * np.abs(ref[net:]).max()
    assert (np.abs(gn - ref[net:]) <= bar).all() and (np.abs(gnz - ref[net:]) <= bar).all()
