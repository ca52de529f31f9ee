"""Exporting a list changes nothing but the caller's arrays, whatever the number of atoms and the
capacities: a row of capacity entries may be longer than all other arrays of a small system."""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import lists_equal, make_system, say

pytestmark = pytest.mark.gpu


# (radial, angular) capacities on both sides of each other and of whole 16-entry segments
@pytest.mark.parametrize("n_atoms,caps", [(1, (160, 96)), (11, (160, 96)), (17, (160, 96)), (21, (200, 161)),
                                          (100, (4096, 4096)), (100, (120, 4096)), (250, (97, 160)), (257, (512, 81))])
def test_export_leaves_the_system(n_atoms, caps):
    say(f"case: {n_atoms} atoms, capacities {caps}, lists exported within a thermostatted run")
    hp, params = I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0)
    at = I.fcc_box(5 if n_atoms > 256 else 4, 0.08, 3)
    rng = np.random.default_rng(n_atoms)
    keep = np.sort(rng.choice(at.n, n_atoms, replace=False))
    at = I.Atoms(x=np.ascontiguousarray(at.x[keep]), types=np.zeros(n_atoms, np.int32), box=at.box,
                 masses=at.masses, v=rng.normal(0.0, 2e-3, (n_atoms, 3)))
    out = []
    for export in (False, True):
        s = make_system(at, hp, params, cap_radial=caps[0], cap_angular=caps[1], skin=0.2)
        s.set_deterministic(True)
        chain = n_atoms > 1
        if chain:
            s.set_thermostat(300.0, tau=20.0, chain=3)
            s.step(2, rebuild_every=0, skin=0.2)
        res = [s.compute(per_atom=True)]
        if export:
            x, _, _ = s.get_state()
            for which, cut in [(0, 6.2), (1, 5.2)]:
                s2 = make_system(I.Atoms(x=x, types=at.types, box=at.box, masses=at.masses), hp, params,
                                 cap_radial=caps[0], cap_angular=caps[1], skin=0.2)
                off, idx = s2.export_neighbors(which)
                cnt, oidx = oracle.neighbors(x, at.box, cut, cap=512)
                ok, msg = lists_equal(off, idx, cnt, oidx)
                assert ok, (which, msg)
                s.export_neighbors(which)
        res.append(s.compute(per_atom=True))
        if chain:
            res.append(s.get_thermostat())
            s.step(2, rebuild_every=0, skin=0.2)
            res.append(s.get_thermostat())
        res.append(s.get_state()[:2])
        out.append(res)
    for a, b in zip(*out):
        for p, q in zip(a, b):
            assert np.array_equal(p, q)
