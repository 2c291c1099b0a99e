"""GPU parity of geek_quantile_buckets' sample sort with the oracle, bit for
bit: sizes around one cell, several sample chunks and groups of tables; values
that crowd a cell's slots (exact comparison sort), that fill whole cells (radix
ranks), that lie in a narrow band or have heavy tails."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def _check(X, A, t, name):
    api = gpu_api()
    announce(f"quantile cells {name} n={len(X)} d={X.shape[1]} m={len(A)} t={t}")
    mem, off, bof = oracle.quantile_buckets(X, A, t)
    gm, go, gb = api.quantile_buckets(cuda(X), cuda(A), t)
    assert np.array_equal(host_u32(go), off)
    assert np.array_equal(host_u32(gb), bof)
    assert np.array_equal(host_u32(gm), mem)
    gm2, _, none = api.quantile_buckets(cuda(X), cuda(A), t, want_bucket_of=False)
    assert none is None and np.array_equal(host_u32(gm2), mem)


@pytest.mark.parametrize("n,d,m,t", [
    (1, 3, 2, 1), (65, 1, 9, 7), (3000, 17, 3, 11), (3001, 16, 8, 5), (8192, 15, 2, 900), (8193, 33, 2, 3),
    (50_001, 7, 41, 1000), (300_007, 5, 2, 64), (5_000_011, 2, 1, 2_000),
])
def test_quantile_sizes(n, d, m, t):
    g = np.random.default_rng(n)
    _check(g.normal(size=(n, d)).astype(np.float32), g.normal(size=(m, d)).astype(np.float32), t, "sizes")


@pytest.mark.parametrize("kind", ["equal", "two", "hundred", "runs", "pairs", "band", "tails", "sorted"])
def test_quantile_value_patterns(kind):
    g = np.random.default_rng(4)
    n = 40_000
    v = {
        "equal": np.zeros(n),                                   # one value: every cell but one empty
        "two": g.integers(0, 2, n),
        "hundred": g.integers(0, 100, n),                       # 400 of each value
        "runs": g.integers(0, 1000, n),                         # 40 of each: crowded slots
        "pairs": np.repeat(g.normal(size=n // 2), 2),           # exact ties in pairs
        "band": 1e6 + g.integers(0, 4000, n) / 4.0,             # far from zero, narrow
        "tails": g.standard_cauchy(n) ** 3,
        "sorted": np.arange(n) - n / 2,                         # ids of a bucket are consecutive
    }[kind]
    X = np.stack([v, g.normal(size=n)], axis=1).astype(np.float32)
    A = np.array([[1, 0], [-1, 0], [0.5, 0.25]], np.float32)
    _check(X, A, 37, kind)      # buckets of 1,081: ranked in LDS
    _check(X, A, 6, kind)       # buckets of 6,667: sorted by bucket
