"""GPU parity at the sizes where small calls take a path of their own: tables
bucketized by one workgroup (up to 2,048 objects), SSE and radii of one block
of rows (up to 4,096 rows and 2,048 clusters), and the next sizes up."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 65, 511, 513, 2047, 2048, 2049])
@pytest.mark.parametrize("kw,alphabet", [(1, 1), (1, 40), (2, 3), (3, 2**31), (4, 7)])
def test_small_tables(n, kw, alphabet):
    api = gpu_api()
    g = np.random.default_rng(n * 5 + kw)
    T = 3
    keys = g.integers(0, alphabet, size=(T, n, kw)).astype(np.uint32)
    announce(f"bucketize small n={n} kw={kw} alphabet={alphabet}")
    for want in (True, False):
        mem, off, nb, bof = api.bucketize(cuda(keys), n, T, kw, n * kw, kw, want_bucket_of=want)
        assert (bof is not None) == want
        for t in range(T):
            rm, ro, rb = oracle.bucketize(keys[t].astype(np.int64))
            assert int(nb[t]) == len(ro) - 1
            assert np.array_equal(host_u32(mem[t]), rm)
            assert np.array_equal(host_u32(off[t])[:len(ro)], ro)
            if want:
                assert np.array_equal(host_u32(bof[t]), rb)


def test_small_tables_rows_of_a_wider_matrix():
    # band layout: all tables' words in one row, rows wider than the bands
    api = gpu_api()
    g = np.random.default_rng(3)
    n, T, kw, ld = 1500, 5, 3, 19
    sig = g.integers(0, 4, size=(n, ld)).astype(np.uint32)
    announce("bucketize small bands")
    mem, off, nb, bof = api.bucketize(cuda(sig), n, T, kw, kw, ld)
    for t in range(T):
        rm, ro, rb = oracle.bucketize(sig[:, t * kw:(t + 1) * kw].astype(np.int64))
        assert int(nb[t]) == len(ro) - 1
        assert np.array_equal(host_u32(mem[t]), rm) and np.array_equal(host_u32(off[t])[:len(ro)], ro)
        assert np.array_equal(host_u32(bof[t]), rb)


@pytest.mark.parametrize("n,k", [(1, 1), (31, 3), (33, 33), (4095, 5), (4096, 2048), (4096, 2049), (4097, 7),
                                 (8191, 40), (8209, 4097)])
def test_sse_and_radius_sizes(n, k):
    api = gpu_api()
    g = np.random.default_rng(n + k)
    X = g.normal(size=(n, 3)).astype(np.float32)
    ids = g.integers(0, n, size=k)
    so, sm = np.arange(k + 1, dtype=np.uint32), ids.astype(np.uint32)
    announce(f"sse n={n} k={k}")
    C = oracle.centroids(X, so, sm)
    a, dist = oracle.assign_euclid(X, C)
    for prec in (0, 1):
        out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, prec)
        assert np.array_equal(out["assign"].cpu().numpy(), a)
        assert out["sse"].item() == oracle.sse(dist)
        assert np.array_equal(out["radius"].cpu().numpy(), oracle.radius(dist, a, k))
        again = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, prec, want_radius=False, want_dist=False)
        assert again["sse"].item() == oracle.sse(dist)


@pytest.mark.parametrize("n,T", [(2049, 1), (4096, 2), (4097, 2), (12289, 40), (20001, 128), (40000, 128), (33000, 256)])
def test_partition_chunk_sizes(n, T):
    # workgroups of the first partition pass take 4,096, 8,192 or 16,384 ids
    api = gpu_api()
    g = np.random.default_rng(n + T)
    keys = g.integers(0, 90, size=(T, n, 4)).astype(np.uint32)
    keys[:, :, 2:] = 0
    announce(f"bucketize chunks n={n} T={T}")
    mem, off, nb, bof = api.bucketize(cuda(keys), n, T, 4, n * 4, 4)
    for t in {0, T // 2, T - 1}:
        rm, ro, rb = oracle.bucketize(keys[t].astype(np.int64))
        assert int(nb[t]) == len(ro) - 1
        assert np.array_equal(host_u32(mem[t]), rm) and np.array_equal(host_u32(off[t])[:len(ro)], ro)
        assert np.array_equal(host_u32(bof[t]), rb)


@pytest.mark.parametrize("n,k", [(4097, 4096), (12288, 4096), (12289, 4097), (20011, 1)])
def test_sse_beside_radii(n, k):
    api = gpu_api()
    g = np.random.default_rng(n + k)
    X = g.normal(size=(n, 3)).astype(np.float32)
    so, sm = np.arange(k + 1, dtype=np.uint32), g.integers(0, n, size=k).astype(np.uint32)
    announce(f"sse beside radii n={n} k={k}")
    a, dist = oracle.assign_euclid(X, oracle.centroids(X, so, sm))
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 1)
    assert np.array_equal(out["assign"].cpu().numpy(), a)
    assert out["sse"].item() == oracle.sse(dist)
    assert np.array_equal(out["radius"].cpu().numpy(), oracle.radius(dist, a, k))


@pytest.mark.parametrize("d", [1, 7, 31, 33, 64, 65, 127, 129, 255, 256])
def test_hash_norms_of_ragged_depths(d):
    # eight lanes share a projection row's norm: depths that leave some of them short
    api = gpu_api()
    g = np.random.default_rng(d)
    n, m, L, w = 300, 5, 13, 3.0
    X = g.normal(size=(n, d)).astype(np.float32)
    A, b = g.normal(size=(m * L, d)).astype(np.float32), (g.random(m * L) * w).astype(np.float32)
    announce(f"hash norms d={d}")
    codes = oracle.e2lsh_codes(X, A, b, w)
    keys, _ = api.hash_dense(cuda(X), cuda(A), cuda(b), m, L, w)
    mem, off, nb, bof = api.bucketize(keys, n, L, 4, n * 4, 4)
    for t in range(L):
        rm, ro, rb = oracle.bucketize(codes[:, t * m:(t + 1) * m])
        assert int(nb[t]) == len(ro) - 1
        assert np.array_equal(host_u32(mem[t]), rm) and np.array_equal(host_u32(off[t])[:len(ro)], ro)
