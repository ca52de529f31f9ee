"""The bfloat16 network at each lane count of the force kernel, one and two species, against the
oracle's bfloat16 model (the same rounding points).

An element within FP32 error of a rounding boundary may round the other way: a center's U then
moves by at most one step, 2^-7 |q~_v|, of one descriptor times sum_mu |w1_mu W0_mu,v|, the
bound of |dU/dq~_v|; two such elements in one center are allowed for. The mean over centers and
the energy per atom stay at FP32 level (2e-6 eV), forces within 5e-3 eV/A: the bars of the
4,000-atom case.
"""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


# force lanes: 16, 8, 4, 4, 2, 1
@pytest.mark.parametrize("cells,species", [(6, 1), (6, 2), (13, 1), (13, 2), (17, 1), (21, 2), (24, 1), (24, 2), (31, 1)])
def test_bf16_against_the_bf16_oracle(cells, species):
    hp = I.HParams(n_types=species)
    params = I.random_model(hp, 2 + species)
    at = I.fcc_box(cells, 0.05, 8)
    at.types = np.random.default_rng(9).integers(0, species, at.n).astype(np.int32)
    at.masses = np.full(species, I.CU_MASS_AMU)
    say(f"case: bf16 network, {at.n} atoms, {species} species")
    s = make_system(at, hp, params)
    E, W, F, U = s.compute(precision="bf16", per_atom=True)
    s.set_deterministic(True)
    Ed, Wd, Fd, Ud = s.compute(precision="bf16", per_atom=True)
    m = oracle.Model.from_hparams(hp, params)
    Eb, Wb, Ub, Fb = oracle.evaluate(m, at.x, at.types, at.box, bf16=True)
    off = hp.offsets()
    sigma, W0, w1 = (params[slice(*off[k])] for k in ("sigma", "W0", "w1"))
    slope = np.abs(w1[:, None] * W0.reshape(hp.n_hidden, hp.n_desc)).sum(0)
    sample = np.random.default_rng(1).choice(at.n, min(at.n, 2000), replace=False)
    q = np.abs(oracle.descriptors(m, at.x, at.types, at.box, sample) * sigma).max(0)
    bound = 2.0 * (2.0 ** -7 * q * slope).max()
    du = np.abs(U - Ub)
    say(f"  max|dU|={du.max():.2e} (bound {bound:.2e}) mean|dU|={du.mean():.2e} max|dF|={np.abs(F - Fb).max():.2e}")
    assert du.mean() < 2e-6 and abs(E - Eb) / at.n < 2e-6
    assert du.max() < bound and np.abs(F - Fb).max() < 5e-3
    assert Ed == E and np.array_equal(Wd, W) and np.array_equal(Ud, U) and np.abs(Fd - F).max() < 1e-6
