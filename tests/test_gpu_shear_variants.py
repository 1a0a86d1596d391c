"""Every shear variant against the first one and the oracle where their code
differs: lines of up to 64, 65 to 128 and more than 128 cells (kernels of
their own for the variants with conditional stores), copied and periodic
ghosts, the three storages, and values below the smallest normal FP32 number
(the tails of a cold plasma), where halved slopes are rounded."""
import numpy as np
import pytest

from paper_2504_21450_amd import binding as B
from paper_2504_21450_amd import workloads as W
from gpuhelp import compare_states, gpu_partition, need_gpu, print_case, run_oracle
from statehelp import random_state

pytestmark = pytest.mark.gpu
TOL64 = 1e-12


def steps(w, storage, variant, neighbours, nsteps=2):
    p = gpu_partition(w, storage=storage)
    if variant is not None:
        p.set_variant(variant)
    for _ in range(nsteps):
        if neighbours:
            p.fill_ghosts_from([p] * 27)
        else:
            p.fill_ghosts()
        p.step(w.dt)
    return p.export(), p.variants()[1]


@pytest.mark.parametrize("storage", [B.VL_F64, B.VL_F32, B.VL_BF16])
@pytest.mark.parametrize("n,order", [((58, 3, 4), (0, 1, 2)), ((59, 3, 3), (2, 1, 0)), ((4, 122, 3), (0, 1, 2)),
                                     ((3, 123, 3), (1, 0, 2)), ((3, 3, 250), (2, 0, 1))])
def test_variants_on_lines_of_every_kernel(n, order, storage):
    """Extents of 64, 65, 128, 129 and 256 cells with their ghost cells, as a
    first, second and last shear; blocks come and go, so segments and gaps
    take every length."""
    need_gpu()
    nblk = (2, 3, 2)
    st = random_state(n, nblk, 83, density=0.4, zero_frac=0.05)
    w = W.Workload("variants", n, (5.0, 7.0, 5.0), nblk, (-4.0, -6.0, -4.0), (1.0,) * 3, 1.0, 2, 2.5e-10, 0,
                   B.VL_F64, order, *st)
    print_case("variants on %s cells, order %s, storage %d" % (n, order, storage))
    o, _ = run_oracle(w, 2)
    want = o.export_local()
    for neighbours in (False, True):
        first, nvar = steps(w, storage, None, neighbours)
        if storage == B.VL_F64:
            compare_states(first, want, TOL64)
        for v in range(nvar):
            got, _ = steps(w, storage, v, neighbours)
            assert all(np.array_equal(a, b) for a, b in zip(got, first)), (v, neighbours)


@pytest.mark.parametrize("storage,scale", [(B.VL_F32, 1e-37), (B.VL_F32, 1e-40), (B.VL_BF16, 1e-37), (B.VL_BF16, 1e-38),
                                           (B.VL_F64, 1e-307), (B.VL_F64, 1e-310), (B.VL_F32, 3e38), (B.VL_F64, 1e308)])
def test_variants_at_the_ends_of_the_range(storage, scale):
    """Values around the smallest normal number and up to the largest: all
    variants give the same bits."""
    need_gpu()
    n, nblk = (24, 9, 8), (2, 3, 2)
    st = random_state(n, nblk, 84, density=0.6, zero_frac=0.05, scale=scale)
    w = W.Workload("ends", n, (9.0, 13.0, 9.0), nblk, (-4.0, -6.0, -4.0), (1.0,) * 3, 1.0, 1, 0.0, 0,
                   B.VL_F64, (0, 1, 2), *st)
    print_case("variants, storage %d, values up to %g" % (storage, scale))
    first, nvar = steps(w, storage, None, False)
    assert np.all(np.isfinite(first[2])) and first[2].any()
    for v in range(nvar):
        got, _ = steps(w, storage, v, False)
        assert all(np.array_equal(a, b) for a, b in zip(got, first)), v
