"""Evaluation with several lanes to a center: system sizes on both sides of every change of
the lane counts (N L <= 131072, L = 16, 8, 4, 2, 1; four lanes in the force kernel up to
49,152 and from 65,537 to 98,304 atoms) and of the workgroup tiles, against the FP64 oracle.

Bars are the FP32 path's stated ones (per-atom energy 1e-6 eV, forces 1e-4 eV/A, virial
1e-6 eV per atom and component); the deterministic form sums the same pair terms in another
order, so its forces may differ by FP32 roundings of a few eV/A-sized partial sums (1e-6 eV/A)
and its energy and virial not at all.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import make_system, say

pytestmark = pytest.mark.gpu


def _box(n_atoms, species, seed):
    """An FCC box thinned at random to n_atoms."""
    cells = 4
    while 4 * cells ** 3 < n_atoms:
        cells += 1
    at = I.fcc_box(cells, 0.08, seed)
    rng = np.random.default_rng(seed + 1)
    keep = np.sort(rng.choice(at.n, size=n_atoms, replace=False))
    at.x = np.ascontiguousarray(at.x[keep])
    at.types = np.ascontiguousarray(rng.integers(0, species, n_atoms).astype(np.int32))
    at.masses = np.full(species, I.CU_MASS_AMU)
    return at


@pytest.mark.parametrize("n_atoms", [1, 17, 255, 4001, 8192, 8193, 16384, 16385, 32769, 49153, 65536, 65537, 98305])
@pytest.mark.parametrize("species", [1, 2])
def test_lane_counts_match_oracle(n_atoms, species):
    say(f"case: {n_atoms} atoms, {species} species, default and deterministic")
    hp = I.HParams(n_types=species)
    params = I.random_model(hp, 3 + species)
    at = _box(n_atoms, species, 70 + n_atoms % 7)
    s = make_system(at, hp, params)
    E, W, F, U = s.compute(per_atom=True)
    s.set_deterministic(True)
    Ed, Wd, Fd, Ud = s.compute(per_atom=True)
    m = oracle.Model.from_hparams(hp, params)
    Eo, Wo, Uo, Fo = oracle.evaluate(m, at.x, at.types, at.box)
    assert np.abs(U - Uo).max() < 1e-6 and abs(E - Eo) / at.n < 1e-6
    assert np.abs(F - Fo).max() < 1e-4 and np.abs(W - Wo).max() / at.n < 1e-6
    assert Ed == E and np.array_equal(Wd, W) and np.array_equal(Ud, U)
    assert np.abs(Fd - F).max() < 1e-6


@pytest.mark.parametrize("n_atoms, species, surrogate", [(131072, 2, False), (131073, 1, False), (131073, 2, False),
                                                        (65537, 2, True)])
def test_two_lanes_in_large_systems(n_atoms, species, surrogate):
    """The force kernel's two lanes beside one lane in the descriptor kernel, and the largest
    size that keeps one."""
    say(f"case: {n_atoms} atoms, {species} species, surrogate {surrogate}")
    hp = I.SURROGATE_SHORTER_HPARAMS if surrogate else I.FULL_HPARAMS
    hp = dataclasses.replace(hp, n_types=species, zbl_z=(29.0,) * species)
    params = I.random_model(hp, 3 + species)
    at = _box(n_atoms, species, 71)
    s = make_system(at, hp, params)
    E, W, F, U = s.compute(per_atom=True)
    s.set_deterministic(True)
    Ed, Wd, Fd, Ud = s.compute(per_atom=True)
    Eo, Wo, Uo, Fo = oracle.evaluate(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box)
    assert np.abs(U - Uo).max() < 1e-6 and abs(E - Eo) / at.n < 1e-6
    assert np.abs(F - Fo).max() < 1e-4 and np.abs(W - Wo).max() / at.n < 1e-6
    assert Ed == E and np.array_equal(Wd, W) and np.array_equal(Ud, U)
    assert np.abs(Fd - F).max() < 1e-6


@pytest.mark.parametrize("n_atoms", [300, 9000, 20000, 40000])
def test_surrogate_lane_counts(n_atoms):
    """The l <= 2 shape (slot 1) at each lane count."""
    say(f"case: {n_atoms} atoms, surrogate")
    hp, params = I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0)
    shp = I.SURROGATE_SHORTER_HPARAMS
    sp = I.surrogate_from_teacher(hp, params, shp, 1)
    at = _box(n_atoms, 1, 91)
    s = make_system(at, hp, params, shp, sp)
    E, W, F, U = s.compute(slot=1, per_atom=True)
    Eo, Wo, Uo, Fo = oracle.evaluate(oracle.Model.from_hparams(shp, sp), at.x, at.types, at.box)
    assert np.abs(U - Uo).max() < 1e-6 and np.abs(F - Fo).max() < 1e-4 and np.abs(W - Wo).max() / at.n < 1e-6
