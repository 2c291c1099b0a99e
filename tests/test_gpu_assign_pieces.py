"""GPU parity of the float32 assignment pass, whose values go to the matrix
cores as two float16 pieces, with the oracle, bit for bit: widths around the
matrix step, rows and seeds of very different magnitudes, values whose low
pieces are subnormal or zero, and near-duplicate seeds that need the rescan."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api

pytestmark = pytest.mark.gpu


def _check(X, so, sm, prec, name):
    api = gpu_api()
    k = len(so) - 1
    announce(f"assign pieces {name} n={len(X)} d={X.shape[1]} k={k} prec={prec}")
    C = oracle.centroids(X, so, sm)
    a, dist = oracle.assign_euclid(X, C)
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, prec)
    assert np.array_equal(out["centroids"].cpu().numpy(), C)
    assert np.array_equal(out["assign"].cpu().numpy(), a)
    assert np.array_equal(out["dist"].cpu().numpy(), dist)
    assert out["sse"].item() == oracle.sse(dist)
    return out["counters"].cpu().numpy()


def _seeds(n, k, g):
    sizes = g.integers(1, 4, size=k)
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    sm = np.concatenate([np.sort(g.choice(n, size=s, replace=False)) for s in sizes]).astype(np.uint32)
    return so, sm


@pytest.mark.parametrize("n,d,k", [(129, 1, 5), (300, 7, 33), (257, 9, 64), (500, 33, 65), (300, 65, 129),
                                   (260, 127, 31), (300, 129, 97), (200, 256, 200)])
def test_pieces_widths(n, d, k):
    g = np.random.default_rng(n + d)
    X = g.normal(size=(n, d)).astype(np.float32) * 10
    so, sm = _seeds(n, k, g)
    for prec in (0, 1):
        _check(X, so, sm, prec, "widths")


@pytest.mark.parametrize("kind", ["rows", "columns", "tiny", "large", "mixed", "integers", "zeros"])
def test_pieces_magnitudes(kind):
    g = np.random.default_rng(8)
    n, d, k = 700, 40, 90
    X = g.normal(size=(n, d))
    if kind == "rows":
        X *= 10.0 ** g.uniform(-12, 6, size=(n, 1))
    elif kind == "columns":
        X *= 10.0 ** g.uniform(-9, 3, size=(1, d))
    elif kind == "tiny":
        X *= 1e-36
    elif kind == "large":
        X *= 3e17
    elif kind == "mixed":
        X[::3] *= 1e-20
        X[1::3] *= 1e12
    elif kind == "integers":
        X = np.rint(X * 1000)
    elif kind == "zeros":
        X[::2] = 0.0
    X = X.astype(np.float32)
    so, sm = _seeds(n, k, g)
    for prec in (0, 1):
        _check(X, so, sm, prec, kind)


@pytest.mark.parametrize("d", [24, 100, 200])
def test_pieces_near_duplicates_rescan(d):
    # thirty seeds within rounding of each other far from the origin: more
    # candidates than a first-pass window, so the rescan and float64 decide
    g = np.random.default_rng(d)
    base = g.uniform(-50, 50, size=d)
    X = (base + g.normal(size=(900, d)) * 0.02).astype(np.float32)
    X[450:] += 25.0
    so, sm = _seeds(900, 60, g)
    ctr = [_check(X, so, sm, prec, "near duplicates") for prec in (0, 1)]
    assert ctr[1][1] + ctr[1][2] > 0  # not settled by the bf16 pass alone
