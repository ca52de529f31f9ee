"""The allocation-free call queues the list build and the evaluation before it knows that the
state is good: a configuration of nothing but bad values is refused, and at an ordinary cost."""
import time

import numpy as np
import pytest
import torch

from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd import nep
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["x", "all"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_a_bad_configuration_costs_what_a_good_one_does(what, precision):
    model = nep.NEPModel(I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0))
    at = I.fcc_box(17, 0.05, 5)   # 19,652 atoms, most of what the fixed scratch holds
    t = torch.tensor(at.types, dtype=torch.int32, device="cuda:0")
    x = torch.tensor(at.x, device="cuda:0")
    bad = x.clone()
    if what == "x":
        bad[:, 0] = float("nan")
    else:
        bad[:] = float("inf")
    F = torch.full((at.n, 3), 7.0, dtype=torch.float64, device="cuda:0")

    def call(pos):
        torch.cuda.synchronize()
        start = time.perf_counter()
        try:
            nep.compute_energy_forces_virial_noalloc(model, pos, t, at.box, precision=precision, forces=F)
            return None, time.perf_counter() - start
        except nep.NEPError as e:
            return e, time.perf_counter() - start

    say(f"case: 19,652 atoms, {what} not finite, {precision}")
    good = []
    for _ in range(3):
        e, dt = call(x)
        assert e is None
        good.append(dt)
    F[:] = 7.0
    e, dt = call(bad)
    say(f"  good {1e3 * min(good):.2f} ms, bad {1e3 * dt:.2f} ms")
    assert e is not None and e.status == -5 and bool((F == 7.0).all())
    # the same work on another arrangement of the atoms; all in one place takes over a thousand times as long
    assert dt < 20.0 * max(good)
