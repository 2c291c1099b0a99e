"""GPU parity of geek_silk_seeds where one job has far more SILK tables than
(table, object) entries: the tables still run in batches that a launch holds."""

import numpy as np
import pytest

import oracle
from workloads import key_words
from workloads.gen import STREAM_SILK

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def test_silk_more_tables_than_a_batch():
    api = gpu_api()
    n, T, K, LS, delta = 6, 3, 1, 16_500, 2
    keys = np.array([[0, 0, 1], [0, 0, 1], [0, 1, 1], [1, 1, 0], [1, 1, 0], [1, 2, 0]], np.int64)
    silk = key_words((LS + 1) * K, 5, STREAM_SILK)
    offs, mem = [0], []
    for mm, oo, _ in oracle.bucketize_tables(keys, 1, T):
        mem.append(mm)
        offs.extend((oo[1:].astype(np.int64) + offs[-1]).tolist())
    ro, rm, info = oracle.silk_seeds(np.asarray(offs, np.int64), np.concatenate(mem), K, LS, delta, silk)
    announce(f"silk tiny n={n} T={T} L={LS} ref k={len(ro) - 1}")
    words = cuda(np.ascontiguousarray(keys.T).astype(np.uint32))
    bm, bo, bn, _ = api.bucketize(words, n, T, 1, n, 1, want_bucket_of=False)
    so, sm, ctr = api.silk_seeds(bm, bo, bn, n, T, K, LS, delta, cuda(silk))
    assert np.array_equal(host_u32(so), ro) and np.array_equal(host_u32(sm), rm)
    ctr = ctr.cpu().numpy()
    assert ctr[0] == info["hash_evals"] and ctr[1] == info["pairs_voted"] and ctr[2] == info["multiset"]
