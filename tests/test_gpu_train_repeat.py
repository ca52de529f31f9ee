"""Training gradients are sums in a fixed order: the same inputs give the same bits, at every lane
count, in one and in two stages of the row sums, with rows in every buffer they may lie in, and
with a list scratch too short for the rows of 16 lanes (values there against the oracle, at the
bars of the training gradients)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd.nep import network_params
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


def _system(n_atoms, shape, species, sparse):
    base = I.FULL_HPARAMS if shape == "full" else I.SURROGATE_HPARAMS
    hp = I.HParams(n_types=species, l_max_3b=base.l_max_3b, l_max_4b=base.l_max_4b, n_hidden=base.n_hidden)
    params = I.random_model(hp, 11 + species)
    cells = 4
    while 4 * cells ** 3 < n_atoms:
        cells += 1
    at = I.fcc_box(cells, 0.1, 21, a=9.0) if sparse else I.fcc_box(cells, 0.1, 21)
    rng = np.random.default_rng(22)
    keep = np.sort(rng.choice(at.n, size=n_atoms, replace=False))
    at = I.Atoms(x=np.ascontiguousarray(at.x[keep]), types=rng.integers(0, species, n_atoms).astype(np.int32), box=at.box,
                 masses=np.full(species, I.CU_MASS_AMU))
    caps = {"cap_radial": 16, "cap_angular": 16} if sparse else {}
    return hp, params, at, make_system(at, hp, params, **caps)


@pytest.mark.parametrize("n_atoms", [3, 250, 4000, 4096, 4097, 16384, 40000, 70000])
@pytest.mark.parametrize("shape,species", [("full", 1), ("full", 2), ("surrogate", 1), ("surrogate", 2)])
def test_gradients_repeat(n_atoms, shape, species):
    say(f"case: {shape} shape, {species} species, {n_atoms} atoms, gradients six times")
    hp, params, at, s = _system(n_atoms, shape, species, False)
    rng = np.random.default_rng(4)
    # weights that grow through the box: workgroups' sums so different in size that FP64 sums of
    # them depend on their order
    scale = 10.0 ** (14.0 * at.x[:, 2:] / at.box[2] - 7.0)
    gF = torch.tensor(rng.normal(size=(at.n, 3)) * scale, dtype=torch.float32, device="cuda")
    p32 = torch.tensor(params, dtype=torch.float32, device="cuda")
    th = torch.tensor(network_params(hp, params), dtype=torch.float32, device="cuda")
    first = None
    for k in range(6):
        got = []
        if k % 2:
            s.compute()          # other contents in the buffers that the rows lie in
        s.train_forward_params(0, p32)
        got.append(s.train_backward_params(0, p32, 0.6, gF))
        got.append(s.train_backward(0, th, 0.6, gF))
        got.append(s.train_backward(0, th, 0.6, gF, out=torch.ones_like(th)))
        got.append(s.train_backward_params(0, p32, 0.6, None))
        if first:  # the FP64 sums' last places, left over when their FP32 values are taken off
            got.append(s.train_backward_params(0, p32, 0.6, gF, out=torch.tensor(-first[0], device="cuda")))
            got.append(s.train_backward(0, th, 0.6, gF, out=torch.tensor(-first[1], device="cuda")))
        got = [g.cpu().numpy() for g in got]
        if first is None or len(first) < len(got):
            first = got if first is None else first + got[len(first):]
        for a, b in zip(first, got):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("n_atoms", [17, 700, 4000])
@pytest.mark.parametrize("shape,species", [("full", 1), ("full", 2), ("surrogate", 2)])
def test_short_list_scratch(n_atoms, shape, species):
    say(f"case: {shape} shape, {species} species, {n_atoms} atoms, radial capacity 16")
    hp, params, at, s = _system(n_atoms, shape, species, True)
    rng = np.random.default_rng(5)
    gF = rng.normal(size=(at.n, 3))
    gFt = torch.tensor(gF, dtype=torch.float32, device="cuda")
    p32 = torch.tensor(params, dtype=torch.float32, device="cuda")
    s.train_forward_params(0, p32)
    g = s.train_backward_params(0, p32, 0.6, gFt).cpu().numpy()
    ref = oracle.param_grad(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box, 0.6, gF)
    off = hp.offsets()
    blocks = [slice(*off[k]) for k in ("cR", "cA", "sigma")] + [slice(off["W0"][0], None)]
    for k in blocks:
        bar = 1e-4 * np.abs(ref[k]) + 1e-5 * np.abs(ref[k]).max()
        assert (np.abs(g[k] - ref[k]) <= bar).all()
