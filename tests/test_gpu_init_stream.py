"""A partition made on a stream of its own (which does not wait for the null
stream, where the clears of its workspace run) in memory that held other
values: moments, and values loaded after the creation, are those of the same
partition made with its values on the default stream."""
import numpy as np
import pytest
import torch

from paper_2504_21450_amd import binding as B
from paper_2504_21450_amd import workloads as W
from gpuhelp import gpu_partition, need_gpu, print_case
from statehelp import random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [B.VL_F64, B.VL_BF16])
def test_partition_on_a_stream_of_its_own(storage):
    need_gpu()
    n, nblk = (6, 5, 4), (12, 11, 13)  # more blocks than a chunk of the moments: cells are split
    state = random_state(n, nblk, 31, density=0.8)
    w = W.Workload("stream", n, (200.0,) * 3, nblk, (-24.0, -22.0, -26.0), (1.0,) * 3, 1.0, 1, 0.0, 0,
                   B.VL_F64, (0, 1, 2), *state)
    print_case("partition on a stream of its own, storage %d" % storage)
    ref = gpu_partition(w, storage=storage)
    want = ref.moments(total=False)[:3]
    # the workspace comes from memory that held other values
    junk = torch.full((ref.ws_bytes + 256,), 0xA5, dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()
    del junk
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        values = torch.from_numpy(w.f).to("cuda:0")
        p = B.Partition(w.n, w.nblk, w.dx, w.vmin, w.dv, w.offsets, w.ids, None, storage=storage)
        assert p.stream.cuda_stream == s.cuda_stream
        empty = p.moments(total=False)
        p.load_values(0, int(w.offsets[-1]), values)
        full = p.moments(total=False)
        s.synchronize()
    assert not empty[0].any() and not empty[2].any()
    assert all(torch.equal(a, b) for a, b in zip(full[:3], want))
