"""Systems with words in the pinned host block and without: which have them, and that runs with
every kind of result read through them agree bit for bit."""
import numpy as np
import pytest

from paper_2604_24816_amd import inputs as I
from paper_2604_24816_amd import nep
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _run(s, at):
    s.set_deterministic(True)
    out = []
    for chain in (0, 3):
        s.set_state(at.x, at.types, at.masses, at.v)
        s.build_neighbors(1.0)
        s.set_thermostat(300.0, tau=20.0, chain=chain)
        out += list(s.compute(per_atom=True)) + [s.step(7, thermo_every=3, rebuild_every=4)] + list(s.get_state())
    s.set_thermostat(300.0, chain=0)
    out.append(s.step(8, mts_k=4, thermo_every=4, fallback_rms=1e9, fallback_max=1e9))
    out += list(s.get_state())
    s.compute(slot=0)
    out += [s.surrogate_error(), s.pair_counts()]
    return out


def test_systems_with_and_without_host_words():
    hp, shp = I.FULL_HPARAMS, I.SURROGATE_SHORTER_HPARAMS
    params = I.random_model(hp, 0)
    full, sur = nep.NEPModel(hp, params), nep.NEPModel(shp, I.surrogate_from_teacher(hp, params, shp, 1))
    at = I.fcc_box(4, 0.05, 3)
    at.v = np.random.default_rng(4).normal(0.0, 2e-3, at.x.shape)
    say("case: 258 systems of 256 atoms; the first has host words, the last has none")
    systems = [nep.NEPSystem(full, at.n, at.box, surrogate=sur) for _ in range(258)]
    assert systems[0].uses_host_words() and not systems[-1].uses_host_words()
    for p, q in zip(_run(systems[0], at), _run(systems[-1], at)):
        assert np.array_equal(p, q) if isinstance(p, np.ndarray) else p == q
    say("words of a closed system go to the next")
    systems[0].close()
    last = nep.NEPSystem(full, at.n, at.box, surrogate=sur)
    assert last.uses_host_words()
