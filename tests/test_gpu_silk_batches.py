"""GPU parity of geek_silk_seeds when its tables run in several batches: the
tables of a job of this size are processed two at a time, so three tables take
a batch of two and a batch of one."""

import numpy as np
import pytest

import oracle
from workloads import key_words
from workloads.gen import STREAM_SILK

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def test_silk_tables_in_two_batches():
    api = gpu_api()
    g = np.random.default_rng(2)
    n, T, K, LS, delta = 28_000, 100, 2, 3, 4
    assert 2 * T * n <= 1 << 23 < 3 * T * n
    # clusters of 200 objects; in every table a cluster's objects share a key
    # except one in five
    keys = np.repeat(np.arange(n // 200), 200)[:, None].repeat(T, axis=1).astype(np.int64)
    stray = g.random((n, T)) < 0.2
    keys[stray] = n + g.integers(0, n, size=int(stray.sum()))
    perm = g.permutation(n)
    keys = keys[perm]
    silk = key_words((LS + 1) * K, 5, STREAM_SILK)
    offs, mem = [0], []
    for mm, oo, _ in oracle.bucketize_tables(keys, 1, T):
        mem.append(mm)
        offs.extend((oo[1:].astype(np.int64) + offs[-1]).tolist())
    ro, rm, info = oracle.silk_seeds(np.asarray(offs, np.int64), np.concatenate(mem), K, LS, delta, silk)
    announce(f"silk batches n={n} T={T} L={LS} ref k={len(ro) - 1}")
    words = cuda(np.ascontiguousarray(keys.T).astype(np.uint32))
    bm, bo, bn, _ = api.bucketize(words, n, T, 1, n, 1, want_bucket_of=False)
    so, sm, ctr = api.silk_seeds(bm, bo, bn, n, T, K, LS, delta, cuda(silk))
    assert len(ro) > 2
    assert np.array_equal(host_u32(so), ro) and np.array_equal(host_u32(sm), rm)
    ctr = ctr.cpu().numpy()
    assert ctr[0] == info["hash_evals"] and ctr[1] == info["pairs_voted"] and ctr[2] == info["multiset"]
