"""GPU parity of the blocked rescan (bf16 first pass, 16,384 seeds or more)
with the oracle, bit for bit: near-duplicate seeds in clusters, widths of every
padded depth, rows that need every seed, duplicated seeds whose ties the lowest
index wins, a device-side seed count, and the same jobs in a batched call."""

import numpy as np
import pytest
import torch

import oracle

from .gpu_util import announce, cuda, gpu_api

pytestmark = pytest.mark.gpu


def _problem(n, d, k, clusters, spread, noise, seed):
    g = np.random.default_rng(seed)
    centers = g.uniform(-spread, spread, size=(clusters, d))
    X = (centers[g.integers(0, clusters, size=n)] + noise * g.normal(size=(n, d))).astype(np.float32)
    sm = g.integers(0, n, size=k).astype(np.uint32)  # one member each, rows repeated: duplicate seeds
    return X, np.arange(k + 1, dtype=np.uint32), sm


def _check(out, X, so, sm, rows):
    C = oracle.centroids(X, so, sm)
    a, dist = oracle.assign_euclid(X[rows], C)
    assert np.array_equal(out["assign"].cpu().numpy()[rows], a)
    assert np.array_equal(out["dist"].cpu().numpy()[rows], dist)


@pytest.mark.parametrize("n,d,k,clusters,spread,noise", [
    (1000, 20, 16_384, 30, 50.0, 1.0),
    (1300, 64, 16_447, 7, 50.0, 1.0),     # ragged: a partly filled last group
    (900, 128, 20_001, 300, 50.0, 1.0),
    (700, 200, 16_500, 12, 20.0, 0.5),
    (600, 33, 16_400, 1, 0.0, 1.0),       # no clusters: every group is marked
    (500, 16, 17_000, 2, 1e18, 1e15),     # windows that overflow float32: float64 decides
])
def test_blocked_rescan(n, d, k, clusters, spread, noise):
    api = gpu_api()
    X, so, sm = _problem(n, d, k, clusters, spread, noise, n + d)
    announce(f"assign blocked n={n} d={d} k={k} clusters={clusters}")
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 1)
    rows = np.arange(0, n, max(1, n // 150))
    _check(out, X, so, sm, rows)
    ctr = out["counters"].cpu().numpy()
    assert ctr[0] + ctr[1] + ctr[2] >= n and ctr[0] < n
    ref = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 0)  # float32 first pass: no blocks
    for name in ("assign", "dist", "sse", "radius"):
        assert torch.equal(out[name], ref[name]), name


def test_blocked_rescan_device_seed_count_and_batch():
    api = gpu_api()
    X, so, sm = _problem(800, 40, 16_600, 20, 50.0, 1.0, 5)
    Xg, sog, smg = cuda(X), cuda(so), cuda(sm)
    k = 16_500
    announce("assign blocked k_dev and batch")
    ref = api.assign_euclid(Xg, sog[:k + 1], smg[:k], k, 1)
    kd = torch.tensor([k], dtype=torch.int32, device="cuda")
    got = api.assign_euclid(Xg, sog, smg, 16_600, 1, k_dev=kd)
    for name in ("assign", "dist", "sse"):
        assert torch.equal(ref[name], got[name]), name
    outs, _ = api.assign_euclid_batch([(Xg, sog[:k + 1], smg[:k], k), (Xg, sog[:11], smg[:10], 10)], 1)
    for name in ("assign", "dist", "sse", "radius"):
        assert torch.equal(ref[name], outs[0][name]), name
