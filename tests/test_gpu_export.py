"""The exported state where its scratch is tight: more cells than work items,
empty cells, and an export between steps that changes nothing."""
import numpy as np
import pytest

from paper_2504_21450_amd import binding as B
from gpuhelp import need_gpu, print_case
from statehelp import random_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("storage", [B.VL_F64, B.VL_F32])
@pytest.mark.parametrize("n,density,cap", [((20, 15, 9), 0.0004, 64), ((3, 3, 3), 0.0, 1), ((5, 4, 3), 0.5, None)])
def test_initial_state_comes_back(n, density, cap, storage):
    nblk = (4, 3, 2)
    off, ids, f = random_state(n, nblk, 3, density=density)
    f = f.astype(np.float32).astype(np.float64)
    kw = {} if cap is None else dict(block_capacity=max(cap, off[-1]), ghost_block_capacity=cap)
    print_case("export of %d blocks in %s cells, storage %d" % (off[-1], n, storage))
    p = B.Partition(n, nblk, (6.0, 5.0, 7.0), (-8.0, -6.0, -4.0), (1.0,) * 3, off, ids, f, storage=storage, **kw)
    for _ in range(2):
        got = p.export()
        assert np.array_equal(got[0], off) and np.array_equal(got[1], ids) and np.array_equal(got[2], f)


def test_exports_between_steps_change_nothing():
    n, nblk = (5, 4, 6), (3, 2, 3)
    st = random_state(n, nblk, 31, density=0.35, zero_frac=0.1)
    print_case("steps with and without exports between them")
    p, q = [B.Partition(n, nblk, (6.0, 5.0, 7.0), (-6.0, -4.0, -6.0), (1.0,) * 3, *st, storage=B.VL_BF16,
                        sparse_min=2.5e-10, vbuffer=6) for _ in range(2)]
    cells = np.arange(p.ncell)
    for _ in range(3):
        for s in (p, q):
            s.fill_ghosts()
            s.step(1.0)
        one, two = p.export(), p.export_cells(cells)
        assert all(np.array_equal(a, b) for a, b in zip(one, two))
    assert all(np.array_equal(a, b) for a, b in zip(p.export(), q.export()))
