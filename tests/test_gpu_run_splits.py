"""Deterministic runs do not depend on where their steps are completed: cut into calls or not, with
a thermo row at every step or none, and resumed from a checkpoint on a step at which the lists were
rebuilt, by an early rebuild or by the caller: positions, velocities and chain bit for bit."""
import numpy as np
import pytest

from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu

DT, SKIN = 2.0, 0.35


def _start(ensemble, species=1, cells=5):
    at = I.fcc_box(cells, 0.08, 6)
    hp = I.HParams(n_types=species)
    if species == 2:
        at.types = np.random.default_rng(5).integers(0, 2, at.n).astype(np.int32)
        at.masses = np.array([I.CU_MASS_AMU, 1.4 * I.CU_MASS_AMU])
    at.v = I.maxwell_boltzmann(at, 1500.0, 7)

    def make(state=None, chain=None):
        a = at if state is None else I.Atoms(x=state[0], types=at.types, box=at.box, masses=at.masses, v=state[1])
        s = make_system(a, hp, I.random_model(hp, 0), skin=SKIN)
        s.set_deterministic(True)
        if ensemble == "nvt":
            s.set_thermostat(1200.0, tau=30.0, chain=4)
            if chain is not None:
                s.set_thermostat_state(*chain)
        return s

    return make


def _result(s, ensemble):
    x, v, _ = s.get_state()
    return [x, v] + (list(s.get_thermostat()[:2]) if ensemble == "nvt" else [])


def _equal(a, b):
    return all(np.array_equal(p, q) for p, q in zip(a, b))


@pytest.mark.parametrize("ensemble", ["nve", "nvt"])
@pytest.mark.parametrize("species", [1, 2])
def test_calls_and_rows_do_not_change_the_run(ensemble, species):
    say(f"case: 14 steps in one call, in calls of 4 + 5 + 5, with a row each step, {ensemble}, {species} species")
    make = _start(ensemble, species)
    out = []
    for calls, rows in (((14,), 0), ((4, 5, 5), 0), ((14,), 1), ((1,) * 14, 3)):
        s = make()
        for n in calls:
            s.step(n, dt=DT, rebuild_every=0, skin=SKIN, thermo_every=rows)
        assert s.stats()["list_builds"] > 1
        out.append(_result(s, ensemble))
    for o in out[1:]:
        assert _equal(out[0], o)


@pytest.mark.parametrize("ensemble", ["nve", "nvt"])
@pytest.mark.parametrize("cells", [5, 9])   # 2 and 12 workgroups of atoms
def test_resume_at_an_early_rebuild(ensemble, cells):
    make = _start(ensemble, cells=cells)
    probe = make()
    builds, first = probe.stats()["list_builds"], 0
    while probe.stats()["list_builds"] == builds:
        probe.step(1, dt=DT, rebuild_every=0, skin=SKIN)
        first += 1
        assert first < 200
    say(f"case: resumed at the early rebuild of step {first}, {ensemble}, {4 * cells ** 3} atoms")
    a = make()
    a.step(first + 12, dt=DT, rebuild_every=0, skin=SKIN)
    b = make()
    b.step(first, dt=DT, rebuild_every=0, skin=SKIN)
    x, v, _ = b.get_state()
    c = make((x, v), b.get_thermostat()[:2] if ensemble == "nvt" else None)
    c.step(12, dt=DT, rebuild_every=0, skin=SKIN)
    b.step(12, dt=DT, rebuild_every=0, skin=SKIN)
    assert _equal(_result(a, ensemble), _result(b, ensemble))
    assert _equal(_result(a, ensemble), _result(c, ensemble))


@pytest.mark.parametrize("ensemble", ["nve", "nvt"])
def test_resume_where_the_caller_rebuilt(ensemble):
    say(f"case: 4 steps, lists rebuilt by the caller, 8 steps, against a resumed run, {ensemble}")
    make = _start(ensemble)
    a = make()
    a.step(4, dt=DT, rebuild_every=0, skin=SKIN)
    x, v, _ = a.get_state()
    c = make((x, v), a.get_thermostat()[:2] if ensemble == "nvt" else None)
    a.build_neighbors(SKIN)
    for s in (a, c):
        s.step(8, dt=DT, rebuild_every=0, skin=SKIN)
    assert _equal(_result(a, ensemble), _result(c, ensemble))
