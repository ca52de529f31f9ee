"""Forces of boxes whose nearest neighbours lie inside the ZBL radius, at every lane count of the
small systems: steep FP32 terms, many times the other forces, that partly cancel.

A component rounded once has an error of 2.5e-8 of its size in the mean square (uniform within half
a last place, the size uniform in its logarithm). The bar allows the force four such roundings,
5.1e-8 of the norm: its own, that of the pair sum's distances, and two more.
"""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [4, 6, 10, 13, 15])   # 16 lanes up to 8,192 atoms, 8 up to 16,384
@pytest.mark.parametrize("deterministic", [False, True])
def test_force_error(cells, deterministic):
    hp = I.HParams(zbl_outer=2.5, zbl_z=(29.0,))
    params = I.random_model(hp, 5)
    at = I.fcc_box(cells, 0.08, 11)
    say(f"case: {at.n} atoms, ZBL radius 2.5 A, deterministic {deterministic}")
    s = make_system(at, hp, params)
    s.set_deterministic(deterministic)
    _, W, F, U = s.compute(per_atom=True)
    Eo, Wo, Uo, Fo = oracle.evaluate(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box)
    err = np.linalg.norm(F - Fo) / np.linalg.norm(Fo)
    say(f"  max|F| {np.abs(Fo).max():.1f} eV/A, relative error {err:.2e}")
    assert err < 5.1e-8
