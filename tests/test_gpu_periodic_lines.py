"""A periodic partition's steps run its local lines alone, their ends read
through the period; the same partition given itself as all 27 neighbours
translates copied ghost lines.  Both give the same state bit for bit, with the
same counts of the ghost scheme."""
import numpy as np
import pytest

import oracle
from oracle import OraclePartition
from paper_2504_21450_amd import binding as B
from paper_2504_21450_amd import workloads as W
from gpuhelp import compare_states, need_gpu, print_case
from statehelp import random_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _partition(n, storage, order, density=0.3, seed=5, **kw):
    nblk = (3, 2, 3)
    st = random_state(n, nblk, seed, density=density, zero_frac=0.1)
    return B.Partition(n, nblk, (6.0, 5.0, 7.0), (-6.0, -4.0, -6.0), (1.0, 1.0, 1.0), *st, storage=storage,
                       order=order, sparse_min=2.5e-10, vbuffer=6, **kw)


# extents at the edges of the mask words: 26 + 6 = 32 cells a padded line, the
# line's first or last three bits across a word boundary, the shortest lines
@pytest.mark.parametrize("n,order", [((3, 3, 3), (0, 1, 2)), ((26, 3, 4), (2, 0, 1)), ((27, 4, 3), (1, 0, 2)),
                                     ((3, 28, 5), (0, 1, 2)), ((4, 3, 29), (2, 1, 0)), ((30, 3, 3), (0, 2, 1)),
                                     ((3, 32, 3), (1, 2, 0)), ((58, 3, 3), (0, 1, 2)), ((3, 3, 61), (2, 0, 1)),
                                     ((250, 3, 3), (0, 1, 2))])
@pytest.mark.parametrize("storage", [B.VL_F64, B.VL_F32, B.VL_BF16])
def test_local_lines_equal_copied_ghost_lines_bitwise(n, order, storage):
    for mode in (B.VL_COALESCED, B.VL_PER_SWEEP):
        print_case("lines of %s, order %s, storage %d, mode %d" % (n, order, storage, mode))
        a, b = _partition(n, storage, order), _partition(n, storage, order)
        for k in range(3):
            v = (0, 4, 6)[k]  # conditional and unconditional stores, streamed items
            a.set_variant(v)
            b.set_variant(v)
            a.fill_ghosts()
            b.fill_ghosts_from([b] * 27)
            sa, sb = a.step(1.0, mode, stats=True), b.step(1.0, mode, stats=True)
            assert sa["updated_ps"] == sb["updated_ps"] and sa["read_ps"] == sb["read_ps"]
            assert sa["items"] == sb["items"] and sa["blocks"] == sb["blocks"]
            ca, cb = a.counters(), b.counters()
            for name in ("ring_head", "ring_tail", "cum_upd", "cum_read"):
                assert ca[name] == cb[name], name
            assert ca["run_upd2"] == cb["upd2"]
        assert all(np.array_equal(x, y) for x, y in zip(a.export(), b.export()))


@pytest.mark.parametrize("storage", [B.VL_F64, B.VL_BF16])
def test_changes_between_local_and_copied_lines(storage):
    """Steps of both kinds in one partition, graph replays among them: the same
    state as copied ghost lines throughout (FP64 and BF16 residuals alike)."""
    n, order = (5, 4, 6), (1, 0, 2)
    print_case("both kinds of steps, storage %d" % storage)
    a, b = _partition(n, storage, order), _partition(n, storage, order)
    for k in range(6):
        b.fill_ghosts_from([b] * 27)
        if k % 3 == 2:
            a.fill_ghosts_from([a] * 27)
            a.step(1.0)
        elif k % 3 == 1:
            a.fill_ghosts()
            a.graph_step(1.0)
        else:
            a.fill_ghosts()
            a.step(1.0)
        b.step(1.0)
    assert all(np.array_equal(x, y) for x, y in zip(a.export(), b.export()))


def test_local_lines_need_no_ghost_room():
    """No ghost block is stored, so none has to fit; copied ones do."""
    n, order = (4, 3, 5), (0, 1, 2)
    print_case("room for one ghost block")
    p, q, r = [_partition(n, B.VL_F64, order, ghost_block_capacity=c) for c in (1, 1, None)]
    for _ in range(2):
        for s in (p, r):
            s.fill_ghosts()
            s.step(1.0)
    assert all(np.array_equal(x, y) for x, y in zip(p.export(), r.export()))
    q.fill_ghosts_from([q] * 27)
    assert q.lib.vl_sync(q.h) == B.VL_ERR_CAPACITY


@pytest.mark.parametrize("n", [(2, 4, 3), (3, 1, 5)])
def test_shorter_lines_keep_copied_ghost_cells(n):
    w = W.Workload("random", n, (6.0, 5.0, 7.0), (3, 2, 3), (-6.0, -4.0, -6.0), (1.0, 1.0, 1.0), 1.0, 3,
                   2.5e-10, 6, B.VL_F64, (0, 1, 2), *random_state(n, (3, 2, 3), 9, density=0.4, zero_frac=0.1))
    print_case("lines of %s" % (n,))
    p, o = B.Partition.from_workload(w), OraclePartition.from_workload(w)
    for _ in range(2):
        p.fill_ghosts()
        p.step(1.0)
        o.fill_ghosts()
        o.step(1.0, oracle.COALESCED)
    compare_states(p.export(), o.export_local(), 1e-12)
