"""The acceleration step's block columns at the edges of what a wavefront
holds: velocity meshes of one block and of 64 blocks along an axis, odd and
even numbers of blocks (the columns' stride in LDS), a single block in the
cell, whole-mesh columns, shifts beyond the mesh."""
import numpy as np
import pytest
import torch

from oracle import OraclePartition
from paper_2504_21450_amd import binding as B
from paper_2504_21450_amd import workloads as W
from gpuhelp import compare_states, need_gpu, print_case
from statehelp import random_state

pytestmark = pytest.mark.gpu
QM = 9.58e7


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nblk,density", [((1, 1, 1), 1.0), ((64, 2, 1), 0.3), ((2, 64, 3), 0.2), ((1, 3, 63), 0.3),
                                          ((5, 4, 6), 1.0), ((7, 6, 5), 0.02), ((8, 8, 9), 0.5)])
@pytest.mark.parametrize("order", [(0, 1, 2), (2, 1, 0)])
def test_columns_match_the_oracle(nblk, density, order):
    """Both compute the same parabolas in FP64: values within 1e-12 of the
    largest.  Fields of the last cells push its blocks off the mesh."""
    n = (3, 2, 3)
    dv = (2e4, 3e4, 2.5e4)
    vmin = tuple(-2.0 * nblk[d] * dv[d] for d in range(3))
    st = random_state(n, nblk, 17, density=density, zero_frac=0.2)
    w = W.Workload("random", n, (1e6, 1e6, 1e6), nblk, vmin, dv, 1.0, 1, 2e-10, 6, B.VL_F64, (0, 1, 2), *st)
    rng = np.random.default_rng(3)
    dt, B0 = 0.3 / (QM * 1e-8), 1e-8
    EB = np.concatenate([rng.normal(size=(w.ncell, 3)) * 1e-3, rng.normal(size=(w.ncell, 3)) * 0.6 * B0], 1)
    EB[-2:, :3] *= 40.0 * max(nblk)
    print_case("columns of %s blocks, density %g, order %s" % (nblk, density, order))
    p = B.Partition.from_workload(w)
    o = OraclePartition.from_workload(w)
    for _ in range(2):
        p.accelerate(dt, QM, torch.tensor(EB.reshape(-1), dtype=torch.float64, device="cuda:0"), order=order)
        o.accelerate(dt, QM, EB, order=order)
        compare_states(p.export(), o.export_local(), 1e-12)


def test_a_large_partition_takes_its_cells_in_several_launches():
    """Room for more than 2^24 blocks: a launch takes as many cells as have
    columns for the item array (4,096 with 64 x 64 columns a cell here)."""
    n, nblk = (17, 16, 16), (64, 64, 1)
    st = random_state(n, nblk, 23, density=0.0004, zero_frac=0.2)
    dv = (2e4, 2e4, 2e4)
    w = W.Workload("random", n, (1e6, 1e6, 1e6), nblk, tuple(-2.0 * nblk[d] * dv[d] for d in range(3)), dv, 1.0, 1,
                   2e-10, 6, B.VL_F32, (0, 1, 2), *st)
    rng = np.random.default_rng(5)
    dt = 0.3 / (QM * 1e-8)
    EB = np.concatenate([rng.normal(size=(w.ncell, 3)) * 1e-3, rng.normal(size=(w.ncell, 3)) * 0.6e-8], 1)
    EBd = torch.tensor(EB.reshape(-1), dtype=torch.float64, device="cuda:0")
    print_case("4352 cells, one and two launches a remap")
    p = B.Partition.from_workload(w, block_capacity=1 << 20, ghost_block_capacity=1 << 20)
    q = B.Partition.from_workload(w, block_capacity=1 << 20, ghost_block_capacity=1 << 24)
    p.accelerate(dt, QM, EBd)
    q.accelerate(dt, QM, EBd)
    assert all(np.array_equal(x, y) for x, y in zip(p.export(), q.export()))


@pytest.mark.parametrize("order", [(0, 1, 2), (2, 1, 0)])
def test_a_value_that_is_not_a_number_spreads_as_in_the_oracle(order):
    """A parabola next to a NaN is none: the same values are NaN as in the
    oracle, not only those that take mass from the NaN's own velocity cell.
    Spatial cells without one agree to 1e-12."""
    n, nblk, dv = (3, 2, 3), (5, 4, 6), (2e4, 3e4, 2.5e4)
    off, ids, f = random_state(n, nblk, 29, density=0.7, zero_frac=0.1)
    f = f.copy()
    poisoned = (0, 7, 11)
    for c in poisoned:
        f[64 * (off[c] + 11) + 21] = np.nan
    w = W.Workload("random", n, (1e6, 1e6, 1e6), nblk, tuple(-2.0 * nblk[d] * dv[d] for d in range(3)), dv, 1.0, 1,
                   0.0, 0, B.VL_F64, (0, 1, 2), off, ids, f)
    rng = np.random.default_rng(7)
    dt = 0.3 / (QM * 1e-8)
    EB = np.concatenate([rng.normal(size=(w.ncell, 3)) * 1e-3, rng.normal(size=(w.ncell, 3)) * 0.6e-8], 1)
    print_case("a NaN in three cells, order %s" % (order,))
    p, o = B.Partition.from_workload(w), OraclePartition.from_workload(w)
    p.accelerate(dt, QM, torch.tensor(EB.reshape(-1), dtype=torch.float64, device="cuda:0"), order=order)
    o.accelerate(dt, QM, EB, order=order)
    got, want = p.export(), o.export_local()
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert np.isnan(want[2]).sum() > len(poisoned)
    assert np.array_equal(np.isnan(got[2]), np.isnan(want[2]))
    for c in set(range(w.ncell)) - set(poisoned):
        a, b = (s[2][64 * s[0][c]:64 * s[0][c + 1]] for s in (got, want))
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(b)
