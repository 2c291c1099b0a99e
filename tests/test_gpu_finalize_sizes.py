"""GPU parity of the float64 distances of settled rows on both sides of the
sizes where eight lanes share a row (wide rows, 2^26 values or more), and of the
counters that the workgroups add up."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(1, 70), (255, 70), (257, 70), (262145, 20), (300007, 64), (262143, 256),
                                 (262145, 256), (1000003, 68)])
def test_distances_either_side_of_the_lane_rule(n, d):
    api = gpu_api()
    g = np.random.default_rng(n + d)
    k = 6
    C = (g.normal(size=(k, d)) * 20).astype(np.float32)
    X = (C[g.integers(0, k, size=n)] + g.normal(size=(n, d)).astype(np.float32)).astype(np.float32)
    so = np.arange(k + 1, dtype=np.uint32)
    sm = g.integers(0, n, size=k).astype(np.uint32)
    announce(f"finalize n={n} d={d}")
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 1)
    rows = np.unique(np.concatenate([np.arange(min(n, 700)), np.arange(max(0, n - 700), n), g.integers(0, n, 700)]))
    a, dist = oracle.assign_euclid(X[rows], oracle.centroids(X, so, sm))
    assert np.array_equal(out["assign"].cpu().numpy()[rows], a)
    assert np.array_equal(out["dist"].cpu().numpy()[rows], dist)
    assert int(out["counters"][:3].sum()) == n


@pytest.mark.parametrize("n,d,dup", [(1 << 18, 257 - 1, 1.0), (700001, 100, 0.5), (700001, 100, 0.02)])
def test_many_rows_leave_the_first_pass(n, d, dup):
    # a share of the rows lies at two seeds at once: no single candidate
    api = gpu_api()
    g = np.random.default_rng(n)
    k = 6
    C = (g.normal(size=(k, d)) * 20).astype(np.float32)
    C[1] = C[0]
    lab = np.where(g.random(n) < dup, 0, g.integers(2, k, size=n))
    X = (C[lab] + g.normal(size=(n, d)).astype(np.float32) * 0.1).astype(np.float32)
    X[:k] = C
    so, sm = np.arange(k + 1, dtype=np.uint32), np.arange(k, dtype=np.uint32)
    announce(f"finalize escalations n={n} d={d} share={dup}")
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 1)
    rows = np.unique(np.concatenate([np.arange(500), np.arange(n - 500, n), g.integers(0, n, 500)]))
    a, dist = oracle.assign_euclid(X[rows], oracle.centroids(X, so, sm))
    assert np.array_equal(out["assign"].cpu().numpy()[rows], a)
    assert np.array_equal(out["dist"].cpu().numpy()[rows], dist)
    ctr = out["counters"].cpu().numpy()
    assert int(ctr[:3].sum()) == n and int(ctr[1] + ctr[2]) >= int((lab == 0).sum()) - k
