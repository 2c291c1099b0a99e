"""GPU parity of the Euclidean assignment with the oracle, bit for bit, where
float32 cannot hold the first pass's values: products that overflow with both
signs, so that a row's accumulators are NaN and no comparison with them holds."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api

pytestmark = pytest.mark.gpu


def _check(X, so, sm, prec, name, rows=None):
    api = gpu_api()
    n, k = len(X), len(so) - 1
    announce(f"assign overflow {name} n={n} d={X.shape[1]} k={k} prec={prec}")
    rows = np.arange(n) if rows is None else rows
    C = oracle.centroids(X, so, sm)
    a, dist = oracle.assign_euclid(X[rows], C)
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, prec)
    assert np.array_equal(out["assign"].cpu().numpy()[rows], a)
    assert np.array_equal(out["dist"].cpu().numpy()[rows], dist)
    ctr = out["counters"].cpu().numpy()
    assert ctr[0] + ctr[1] + ctr[2] == n


LARGEST = np.finfo(np.float32).max  # infinite in bf16: its products with both signs sum to NaN


@pytest.mark.parametrize("n,d,k,share,size", [
    (400, 32, 16_400, 1.0, 1e25),       # every row and seed
    (300, 100, 16_384, 1.0, 1e25),
    (500, 16, 17_000, 0.1, 1e25),       # one row in ten, so most groups hold ordinary seeds
    (400, 32, 16_400, 1.0, LARGEST),
    (500, 16, 17_000, 0.1, LARGEST),
    (300, 200, 16_500, 0.2, LARGEST),
    (2_300, 32, 16_400, 1.0, 1e25),
    (2_300, 20, 16_400, 1.0, LARGEST),
    (700, 100, 16_384, 1.0, 1e25),
])
@pytest.mark.parametrize("prec", [1, 2])
def test_marks_of_rows_without_a_bound(n, d, k, share, size, prec):
    g = np.random.default_rng(n + d)
    X = g.normal(size=(n, d))
    big = g.random(n) < share
    X[big] = np.sign(X[big]) * LARGEST if size == LARGEST else X[big] * size
    X = X.astype(np.float32)
    # seeds from the first rows only: a row that is its own seed has products
    # of one sign, whose sum is not NaN
    sm = g.integers(0, n // 4, size=k).astype(np.uint32)
    rows = np.unique(np.concatenate([np.flatnonzero(big)[-60:], np.arange(0, n, 9)]))
    _check(X, np.arange(k + 1, dtype=np.uint32), sm, prec, "marks", rows)
