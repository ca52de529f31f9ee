"""Training gradients on both sides of every change of the lane count of the gradient kernel
(16 lanes to a center up to 4,096 atoms, 4 up to 16,384, then 2, or 4 for the l <= 2 shape)
and for systems of less than one wavefront, against the oracle's FP64 gradient entry by
entry: |g - ref| <= 1e-4 |ref| + 1e-5 max|ref|, the bar of the training gradients (the floor
covers entries whose FP32 error is set by the block's scale)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd.nep import network_params
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


def _box(n_atoms, species, seed):
    """An FCC box thinned at random to n_atoms, at least 4 cells a side."""
    cells = 4
    while 4 * cells ** 3 < n_atoms:
        cells += 1
    at = I.fcc_box(cells, 0.1, seed)
    rng = np.random.default_rng(seed + 1)
    keep = np.sort(rng.choice(at.n, size=n_atoms, replace=False))
    at.x = np.ascontiguousarray(at.x[keep])
    at.types = np.ascontiguousarray(rng.integers(0, species, n_atoms).astype(np.int32))
    at.masses = np.full(species, I.CU_MASS_AMU)
    return at


@pytest.mark.parametrize("n_atoms", [3, 250, 4096, 4097, 16385])
@pytest.mark.parametrize("shape,species", [("full", 1), ("full", 2), ("surrogate", 1)])
def test_gradients_at_lane_counts(n_atoms, shape, species):
    say(f"case: {shape} shape, {species} species, {n_atoms} atoms, gradients of network and coefficients")
    base = I.FULL_HPARAMS if shape == "full" else I.SURROGATE_HPARAMS
    hp = I.HParams(n_types=species, l_max_3b=base.l_max_3b, l_max_4b=base.l_max_4b, n_hidden=base.n_hidden)
    params = I.random_model(hp, 11 + species)
    at = _box(n_atoms, species, 21)
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
    blocks = {k: slice(*off[k]) for k in ("cR", "cA", "sigma")}
    blocks["network"] = slice(net, None)
    for name, k in blocks.items():
        bar = 1e-4 * np.abs(ref[k]) + 1e-5 * np.abs(ref[k]).max()
        assert (np.abs(g[k] - ref[k]) <= bar).all(), name
    bar = 1e-4 * np.abs(ref[net:]) + 1e-5 * np.abs(ref[net:]).max()
    assert (np.abs(gn - ref[net:]) <= bar).all()
