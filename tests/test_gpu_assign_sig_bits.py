"""GPU parity of the bit-plane signature assignment (k * F <= 2^20, k <= 4096)
with the oracle, bit for bit: seed counts around the lanes' mask words and the
sort's powers of two, widths around a wavefront's positions and the planes'
widths, and a position whose values no tried hash can spread."""

import numpy as np
import pytest

import oracle

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def _run(api, sig, so, sm, name):
    n, F = sig.shape
    k = len(so) - 1
    announce(f"assign-sig bits {name} n={n} F={F} k={k}")
    M = oracle.modes(sig, so, sm)
    a, dist = oracle.assign_sig(sig, M)
    out = api.assign_sig(cuda(sig), cuda(so), cuda(sm), k)
    assert np.array_equal(host_u32(out["modes"]), M)
    assert np.array_equal(out["assign"].cpu().numpy(), a)
    assert np.array_equal(out["dist"].cpu().numpy(), dist)
    assert out["sse"].item() == oracle.sse(dist)
    assert np.array_equal(out["radius"].cpu().numpy(), oracle.radius(dist, a, k, euclid=False))
    assert out["counters"].cpu().numpy()[2] == n  # every row met every mode


@pytest.mark.parametrize("n,F,k,alphabet", [
    (65, 64, 1, 50), (67, 1, 3, 2), (130, 63, 33, 20), (129, 65, 128, 1000), (131, 256, 129, 40),
    (97, 511, 300, 30), (97, 512, 300, 30), (61, 513, 1025, 100), (33, 1024, 1024, 5),
    (201, 255, 2048, 2000), (199, 257, 2049, 60), (301, 256, 4096, 10**6),
])
def test_sig_bits_edges(n, F, k, alphabet):
    api = gpu_api()
    g = np.random.default_rng(n + F + k)
    sig = (g.random((n, F)) ** 2 * alphabet).astype(np.uint32) * np.uint32(2654435761)
    sig[: n // 8] = sig[0]  # rows that match a mode in every position
    sig[-1] = 0xFFFFFFFF
    sizes = g.integers(1, 4, size=k)
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    sm = np.concatenate([np.sort(g.choice(n, size=s, replace=False)) for s in sizes]).astype(np.uint32)
    _run(api, sig, so, sm, "edges")


def test_sig_bits_values_no_hash_spreads():
    # for each of the six hashes tried, five values that agree in its nine low
    # bits (the largest bucket count for k = 40 seeds): every try overflows a
    # bucket, and the position's values are found by binary search
    api = gpu_api()
    v = np.arange(1, 20_001, dtype=np.uint32)

    def mixed(seed):
        h = v ^ np.uint32(seed * 0x9E3779B9 & 0xFFFFFFFF)
        for shift, mul in ((16, 0x85EBCA6B), (13, 0xC2B2AE35)):
            h ^= h >> np.uint32(shift)
            h *= np.uint32(mul)
        return h ^ (h >> np.uint32(16))

    values = []
    for seed in range(6):
        low = mixed(seed) & 511
        values += list(v[low == low[100 + seed]][:5])
    values = np.unique(np.asarray(values, np.uint32))
    assert len(values) >= 26
    g = np.random.default_rng(9)
    n, F, k = 400, 70, 40
    sig = g.integers(0, 50, size=(n, F)).astype(np.uint32)
    sig[:, 3] = g.choice(np.concatenate([values, [0, 7, 0xFFFFFFFF]]).astype(np.uint32), size=n)
    sig[:k, 3] = np.resize(values, k)
    so, sm = np.arange(k + 1, dtype=np.uint32), np.arange(k, dtype=np.uint32)  # one member each
    _run(api, sig, so, sm, "search")


@pytest.mark.parametrize("F", [7, 256, 300])
def test_sig_modes_of_small_and_large_seeds(F):
    # modes counted in LDS (up to 48 members) beside ones found by sorting,
    # with ties between values
    api = gpu_api()
    g = np.random.default_rng(F)
    n = 500
    sig = (g.integers(0, 4, size=(n, F)) * 1_000_003).astype(np.uint32)
    sig[3] = 0xFFFFFFFF
    sizes = np.array([1, 48, 49, 2, 300, 47, 64, 1, 1, 500, 3])
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    sm = np.concatenate([np.sort(g.choice(n, size=s, replace=False)) for s in sizes]).astype(np.uint32)
    _run(api, sig, so, sm, "modes")
