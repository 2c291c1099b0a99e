"""GPU parity of small tables (one workgroup each) whose buckets lie around the
size from which they are sorted instead of counted."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [96, 97, 100, 1023, 1025, 2048])
@pytest.mark.parametrize("size", [95, 96, 97, 500])
def test_crowded_small_tables(n, size):
    # table 0: runs of `size` equal keys, table 1: the same shuffled, table 2: one
    # large bucket beside single objects
    api = gpu_api()
    g = np.random.default_rng(n + size)
    run = np.arange(n) // size
    one = np.where(g.permutation(n) < size, 0, 1 + np.arange(n))
    keys = np.stack([run, g.permutation(run), one])[:, :, None].astype(np.uint32)
    announce(f"bucketize crowded n={n} size={size}")
    mem, off, nb, bof = api.bucketize(cuda(keys), n, 3, 1, n, 1)
    mem2, _, _, none = api.bucketize(cuda(keys), n, 3, 1, n, 1, want_bucket_of=False)
    assert none is None
    for t in range(3):
        rm, ro, rb = oracle.bucketize(keys[t].astype(np.int64))
        assert int(nb[t]) == len(ro) - 1
        assert np.array_equal(host_u32(mem[t]), rm) and np.array_equal(host_u32(mem2[t]), rm)
        assert np.array_equal(host_u32(off[t])[:len(ro)], ro)
        assert np.array_equal(host_u32(bof[t]), rb)
