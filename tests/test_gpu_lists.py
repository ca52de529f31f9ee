"""List build at the sizes where its parts change: one-workgroup sort (up to 16,384 atoms in
2,048 cells) against the general one, halo tables from the cell bitmap (up to 262,144 cells)
against sorted candidates, several workgroups per cell, and boxes that mix dimensions of two
and of more cells. Lists are compared with the oracle's bit for bit; forces at the FP32
path's stated bounds."""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import lists_equal, make_system, say

pytestmark = pytest.mark.gpu


def _fcc(nx, ny, nz, drop, seed, box=None):
    """FCC block of nx x ny x nz cells less `drop` random atoms, in its own box or a larger one."""
    n = max(nx, ny, nz)
    x, _ = I.fcc_lattice(n)
    top = np.array([nx, ny, nz]) * I.CU_LATTICE_A
    x = x[(x < top - 1e-9).all(axis=1)]
    rng = np.random.default_rng(seed)
    x = x[np.sort(rng.choice(len(x), len(x) - drop, replace=False))]
    box = top if box is None else np.asarray(box, float)
    x = I.wrap(x + rng.normal(0.0, 0.08, x.shape), box)
    return I.Atoms(x=x, types=np.zeros(len(x), np.int32), box=box, masses=np.array([I.CU_MASS_AMU]))


CASES = {
    "two cells by two by four": dict(nx=4, ny=5, nz=9, drop=3),
    "three cells, 8 workgroups each": dict(nx=6, ny=6, nz=6, drop=0),
    "largest one-workgroup sort": dict(nx=16, ny=16, nz=16, drop=0),
    "first general sort by atoms": dict(nx=16, ny=16, nz=17, drop=1023),
    "stencils of every atom, larger staging": dict(nx=7, ny=7, nz=7, drop=0),
    "cells of 8.0 A": dict(nx=11, ny=11, nz=11, drop=5),
    "general sort by cells": dict(nx=8, ny=8, nz=8, drop=0, box=(100.0, 101.0, 99.0)),
    "sorted halo candidates": dict(nx=10, ny=10, nz=10, drop=17, box=(470.0, 465.0, 460.0)),
}


@pytest.mark.parametrize("name", CASES)
def test_lists_and_forces(name):
    hp, params = I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0)
    at = _fcc(seed=5, **CASES[name])
    say(f"case: {name}, {at.n} atoms, box {at.box.tolist()}")
    s = make_system(at, hp, params)
    for which, cut in [(0, 7.0), (1, 6.0)]:
        off, idx = s.export_neighbors(which)
        cnt, oidx = oracle.neighbors(at.x, at.box, cut)
        ok, msg = lists_equal(off, idx, cnt, oidx)
        assert ok, (which, msg)
    E, W, F, U = s.compute(per_atom=True)
    Eo, Wo, Uo, Fo = oracle.evaluate(oracle.Model.from_hparams(hp, params), at.x, at.types, at.box)
    assert np.abs(U - Uo).max() < 1e-6 and np.abs(F - Fo).max() < 1e-4 and np.abs(W - Wo).max() / at.n < 1e-6
    # every build starts from the cell counts the last one left at zero
    s.build_neighbors(1.0)
    assert s.compute()[0] == E


@pytest.mark.parametrize("n_atoms", [2300, 4400, 4900, 6000])
def test_staged_and_unstaged_stencils(n_atoms):
    """Random atoms in a 30 A box (cells of 7.5 A, stencils of 0.42 n): staged in the smallest
    size, in the largest, in some cells only, and in none."""
    hp, params = I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0)
    rng = np.random.default_rng(n_atoms)
    box = np.array([30.0, 30.5, 29.9])
    at = I.Atoms(x=rng.uniform(0.0, 1.0, (n_atoms, 3)) * box, types=np.zeros(n_atoms, np.int32), box=box,
                 masses=np.array([I.CU_MASS_AMU]))
    say(f"case: {n_atoms} random atoms, lists only")
    s = make_system(at, hp, params, cap_radial=512, cap_angular=512)
    for which, cut in [(0, 7.0), (1, 6.0)]:
        off, idx = s.export_neighbors(which)
        cnt, oidx = oracle.neighbors(at.x, at.box, cut, cap=512)
        ok, msg = lists_equal(off, idx, cnt, oidx)
        assert ok, (which, msg)


def test_rebuild_on_displacement_and_schedule():
    """20 steps with a small skin (0.2 A, early rebuilds) follow the oracle's velocity Verlet."""
    hp, params = I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0)
    at = I.fcc_box(5, 0.08, 6)
    at.v = I.maxwell_boltzmann(at, 1200.0, 7)
    say("case: 20 steps, skin 0.2 A, no schedule: the displacement test alone rebuilds")
    s = make_system(at, hp, params, skin=0.2)
    s.step(20, dt=1.0, rebuild_every=0, skin=0.2)
    x, v, _ = s.get_state()
    m = oracle.Model.from_hparams(hp, params)
    xo, vo, _ = oracle.velocity_verlet(m, at.x, at.v, at.types, at.masses, at.box, 1.0, 20)
    d = x - xo
    d -= at.box * np.round(d / at.box)
    assert np.abs(d).max() < 1e-6 and np.abs(v - vo).max() < 1e-7
    # 1200 K atoms pass 0.1 A within the run, so lists were rebuilt; never more than once a step
    assert 2 <= s.stats()["list_builds"] <= 21
