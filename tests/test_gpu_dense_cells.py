"""List build of cells of more than 256 atoms: the sort takes the cell's keys 256 at a time."""
import numpy as np
import pytest

import oracle
from paper_2604_24816_amd import inputs as I
from tests.gpu_helpers import lists_equal, make_system, min_image_diff, say

pytestmark = pytest.mark.gpu


def _one_cell(n, seed):
    """n atoms, shuffled, in a 7 A cube that lies in one cell (7.5 A) of a 30 A box; 40 elsewhere."""
    rng = np.random.default_rng(seed)
    box = np.array([30.0, 30.0, 30.0])
    x = np.concatenate([7.7 + 7.0 * rng.random((n, 3)), rng.uniform(0.0, 30.0, (40, 3))])
    rng.shuffle(x)
    return I.Atoms(x=x, types=rng.integers(0, 2, len(x)).astype(np.int32), box=box, masses=np.array([50.0, 70.0]),
                   v=rng.normal(0.0, 1e-3, x.shape))


@pytest.mark.parametrize("n", [255, 257, 512, 513, 1300])
def test_lists_and_state_of_a_dense_cell(n):
    say(f"case: {n} atoms in one cell")
    hp = I.HParams(n_types=2)
    params = I.random_model(hp, 1)
    at = _one_cell(n, n)
    out = []
    for _ in range(2):
        s = make_system(at, hp, params, cap_radial=2048, cap_angular=2048)
        s.set_deterministic(True)
        x, v, _ = s.get_state()
        assert np.array_equal(v, at.v) and np.abs(min_image_diff(x, at.x, at.box)).max() < 1e-13
        for which, cut in [(0, 7.0), (1, 6.0)]:
            off, idx = s.export_neighbors(which)
            cnt, oidx = oracle.neighbors(at.x, at.box, cut, cap=2048)
            ok, msg = lists_equal(off, idx, cnt, oidx)
            assert ok, (which, msg)
        out.append(s.compute(per_atom=True))
    # the atoms' order, and with it every sum, is the same whatever order the scatter left
    for a, b in zip(*out):
        assert np.array_equal(a, b)



@pytest.mark.parametrize("n_atoms,shape", [(2049, (2, 2, 2)), (4097, (2, 3, 4)), (9000, (3, 3, 3)), (20000, (4, 4, 4)),
                                           (33000, (5, 4, 4))])
def test_stencils_in_parts(n_atoms, shape):
    """Stencils of 2,049 to about 10,000 atoms, staged in two to six parts (shape: cells a side)."""
    say(f"case: {n_atoms} random atoms in {shape} cells")
    rng = np.random.default_rng(n_atoms)
    box = 7.1 * np.array(shape, float) + np.array([0.2, 0.3, 0.25])
    at = I.Atoms(x=rng.random((n_atoms, 3)) * box, types=np.zeros(n_atoms, np.int32), box=box,
                 masses=np.array([I.CU_MASS_AMU]))
    s = make_system(at, I.FULL_HPARAMS, I.random_model(I.FULL_HPARAMS, 0), cap_radial=3072, cap_angular=3072)
    for which, cut in [(0, 7.0), (1, 6.0)]:
        off, idx = s.export_neighbors(which)
        cnt, oidx = oracle.neighbors(at.x, at.box, cut, cap=3072)
        ok, msg = lists_equal(off, idx, cnt, oidx)
        assert ok, (which, msg)
