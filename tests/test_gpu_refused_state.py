"""A refused state: its positions have replaced the earlier ones, so that nothing may be computed
from the system until a state is accepted; a refused argument leaves the system as it was."""
import numpy as np
import pytest
import torch

from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd import nep
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


def _alloy():
    at = I.fcc_box(4, 0.05, 3)
    rng = np.random.default_rng(4)
    at.types = rng.integers(0, 2, at.n).astype(np.int32)
    at.masses = np.array([60.0, 100.0])
    at.v = rng.normal(0.0, 2e-3, at.x.shape)
    hp = I.HParams(n_types=2)
    return at, hp, I.random_model(hp, 0)


@pytest.mark.parametrize("fault", ["position", "velocity", "species"])
@pytest.mark.parametrize("device", [False, True])
def test_nothing_is_computed_from_a_refused_state(fault, device):
    at, hp, params = _alloy()
    say(f"case: 256 atoms, evaluated, then a state with a bad {fault}, {'device' if device else 'host'} arrays")
    s = make_system(at, hp, params)
    s.set_deterministic(True)
    good = s.compute(per_atom=True)
    s.step(3)
    x, v, t = at.x.copy(), at.v.copy(), at.types.copy()
    if fault == "position":
        x[7, 1] = np.nan
    elif fault == "velocity":
        v[200, 2] = np.inf
    else:
        t[9] = 2
    args = [x, t, at.masses, v]
    if device:
        args = [torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda"), at.masses, torch.tensor(v, device="cuda")]
    with pytest.raises(nep.NEPError) as e:
        s.set_state(*args)
    assert e.value.status == (-4 if fault == "species" else -5)
    theta = torch.tensor(nep.network_params(hp, params), dtype=torch.float32, device="cuda")
    for call in (lambda: s.compute(), lambda: s.compute(precision="fp64"), lambda: s.build_neighbors(1.0),
                 lambda: s.compute(), lambda: s.step(2), lambda: s.get_state(), lambda: s.export_neighbors(0),
                 lambda: s.train_forward(0, theta), lambda: s.train_backward(0, theta, 1.0, None)):
        with pytest.raises(nep.NEPError):
            call()
    say("then the good state again")
    s.set_state(at.x, at.types, at.masses, at.v)
    s.build_neighbors(1.0)
    for a, b in zip(good, s.compute(per_atom=True)):
        assert np.array_equal(a, b)


def test_refused_masses_leave_the_state():
    at, hp, params = _alloy()
    say("case: 256 atoms, masses refused between two halves of a run")
    runs = []
    for bad in (False, True):
        s = make_system(at, hp, params)
        s.set_deterministic(True)
        s.step(2)
        if bad:
            with pytest.raises(nep.NEPError):
                s.set_state(at.x, at.types, [1.0, -1.0])
        s.step(2)
        runs.append(s.get_state())
    assert np.array_equal(runs[0][0], runs[1][0]) and np.array_equal(runs[0][1], runs[1][1])
