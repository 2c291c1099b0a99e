"""GPU parity of geek_quantile_buckets with the oracle, bit for bit: tables whose
tied values go to the radix ranks beside tables that do not, tables in several
groups with a short last one, and more rows than the sample sort takes."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def _check(X, A, t, tables, name):
    api = gpu_api()
    announce(f"quantile groups {name} n={len(X)} d={X.shape[1]} m={len(A)} t={t}")
    mem, off, bof = oracle.quantile_buckets(X, A[tables], t)
    gm, go, gb = api.quantile_buckets(cuda(X), cuda(A), t)
    api.release_workspace()
    for r, p in enumerate(tables):
        assert np.array_equal(host_u32(go[p]), off[r]), p
        assert np.array_equal(host_u32(gb[p]), bof[r]), p
        assert np.array_equal(host_u32(gm[p]), mem[r]), p


@pytest.mark.parametrize("n,share", [(8193, 1.0), (20_000, 0.6), (300_007, 0.1), (300_007, 0.9), (1_000_003, 0.01)])
@pytest.mark.parametrize("t", [3, 700])
def test_tied_tables_beside_untied_ones(n, share, t):
    # rows whose first attribute is zero for a share of them: projections on it
    # alone are tied there, those with the second are not
    g = np.random.default_rng(n)
    X = g.normal(size=(n, 2)).astype(np.float32)
    X[g.random(n) < share, 0] = 0.0
    A = np.array([[1, 0], [0, 1], [-2, 0], [1, 1], [0.5, 0]], np.float32)
    _check(X, A, t, np.arange(5), "ties")


def test_several_groups_of_tables():
    # 21 and 20 tables of 5 10^6 rows
    g = np.random.default_rng(1)
    X = g.normal(size=(5_000_011, 2)).astype(np.float32)
    X[g.random(len(X)) < 0.01, 0] = 0.0
    A = g.normal(size=(41, 2)).astype(np.float32)
    A[[20, 22, 40], 1] = 0.0
    _check(X, A, 3_000, np.array([0, 20, 21, 22, 40]), "groups")


@pytest.mark.parametrize("t", [20_000, 9])
def test_more_rows_than_the_sample_sort_takes(t):
    g = np.random.default_rng(2)
    X = g.normal(size=(24_600_001, 1)).astype(np.float32)
    X[::50] = 0.0
    _check(X, np.array([[1.5]], np.float32), t, np.arange(1), "rows")


@pytest.mark.parametrize("n,t", [(1, 1), (70, 70), (257, 129), (8193, 8193), (30_011, 469), (30_011, 468), (30_016, 469),
                                 (30_017, 469), (100_003, 50_002)])
def test_small_buckets(n, t):
    # buckets around 64 objects, of one and two, in tied and untied tables
    g = np.random.default_rng(n + t)
    X = g.normal(size=(n, 2)).astype(np.float32)
    X[g.random(n) < 0.4, 0] = 0.0
    _check(X, np.array([[1, 0], [0.3, 1]], np.float32), t, np.arange(2), "small buckets")
