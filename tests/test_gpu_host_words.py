"""Flags and results through host words: with and without a block of them (a process has 256;
systems past that copy), and the allocation-free call, whose checks come after everything is
queued: an error leaves the caller's arrays as they were.

The two forms run the same kernels in the same order: sums, deterministic forces and per-atom
energies are equal bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd import nep
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module")
def model():
    return nep.NEPModel(I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0))


def _run(s, at):
    s.set_deterministic(True)
    s.set_state(at.x, at.types, at.masses, at.v)
    s.build_neighbors(1.0)
    out = list(s.compute(per_atom=True)) + [s.step(12, thermo_every=5)] + list(s.get_state()) + [s.stats()]
    errors = []
    bad_x, bad_t = at.x.copy(), at.types.copy()
    bad_x[7, 1], bad_t[9] = np.inf, 1
    for x, t in ((bad_x, at.types), (at.x, bad_t)):
        with pytest.raises(nep.NEPError) as e:
            s.set_state(x, t, at.masses)
        errors.append(str(e.value))
    s.set_state(at.x, at.types, at.masses)
    s.build_neighbors(1.0)
    return out + [s.compute()[0]], errors


def test_systems_past_the_host_words(model):
    at = I.fcc_box(4, 0.05, 3)
    at.v = np.random.default_rng(4).normal(0.0, 2e-3, at.x.shape)
    say("case: 260 systems of 256 atoms, the first and the last compared")
    systems = [nep.NEPSystem(model, at.n, at.box) for _ in range(260)]
    (a, ea), (b, eb) = _run(systems[0], at), _run(systems[-1], at)
    for p, q in zip(a, b):
        assert np.array_equal(p, q) if isinstance(p, np.ndarray) else p == q
    assert ea == eb
    say("overflowing lists, with host words and without")
    small = nep.NEPSystem(model, at.n, at.box, cap_radial=16)
    systems.append(small)
    messages = []
    del systems[1:3]  # two words come free
    for s in (small, nep.NEPSystem(model, at.n, at.box, cap_radial=16)):
        s.set_state(at.x, at.types, at.masses)
        with pytest.raises(nep.NEPError, match="overflow") as e:
            s.build_neighbors(1.0)
        messages.append(str(e.value))
    assert messages[0] == messages[1]


@pytest.mark.parametrize("fault", ["position", "species", "radial", "angular"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_noalloc_error_keeps_outputs(model, fault, precision):
    at = I.fcc_box(4, 0.05, 5)
    x = torch.tensor(at.x, device="cuda:0")
    t = torch.tensor(at.types, dtype=torch.int32, device="cuda:0")
    caps = {}
    if fault == "position":
        x[11, 2] = float("nan")
    elif fault == "species":
        t[255] = -1
    else:
        caps = {"radial": {"cap_radial": 32}, "angular": {"cap_angular": 32}}[fault]
    F = torch.full((at.n, 3), 7.0, dtype=torch.float64, device="cuda:0")
    U = torch.full((at.n,), 8.0, dtype=torch.float64, device="cuda:0")
    say(f"case: allocation-free call, {fault} at fault, {precision}")
    with pytest.raises(nep.NEPError) as e:
        nep.compute_energy_forces_virial_noalloc(model, x, t, at.box, precision=precision, forces=F,
                                                 per_atom_energy=U, **caps)
    want = {"position": "non-finite", "species": "type", "radial": "capacity", "angular": "capacity"}[fault]
    assert want in str(e.value)
    assert bool((F == 7.0).all()) and bool((U == 8.0).all())
    say("then a good configuration through the same scratch")
    x, t = torch.tensor(at.x, device="cuda:0"), torch.tensor(at.types, dtype=torch.int32, device="cuda:0")
    E, W = nep.compute_energy_forces_virial_noalloc(model, x, t, at.box, precision=precision, forces=F,
                                                    per_atom_energy=U)
    s = nep.NEPSystem(model, at.n, at.box)
    s.set_state(at.x, at.types, at.masses)
    s.build_neighbors(1.0)
    Es, Ws, Fs, Us = s.compute(precision=precision, per_atom=True)
    assert E == Es and np.array_equal(W, Ws) and np.array_equal(U.cpu().numpy(), Us)
