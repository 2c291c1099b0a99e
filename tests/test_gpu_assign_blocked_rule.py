"""GPU parity of the bf16 assignment with 16,384 seeds or more with the oracle,
bit for bit, on both sides of the rule that takes the blocked rescan (rows, and
rows x seeds x padded attributes, of all rows on the host and of the unsettled
ones on the device) and past the sizes of its lists."""

import numpy as np
import pytest
import torch

import oracle

from .gpu_util import announce, cuda, gpu_api

pytestmark = pytest.mark.gpu


def _run(X, sm, rows, name):
    api = gpu_api()
    n, k = len(X), len(sm)
    announce(f"assign blocked rule {name} n={n} d={X.shape[1]} k={k}")
    so = np.arange(k + 1, dtype=np.uint32)
    out = api.assign_euclid(cuda(X), cuda(so), cuda(sm), k, 1)
    a, dist = oracle.assign_euclid(X[rows], oracle.centroids(X, so, sm))
    assert np.array_equal(out["assign"].cpu().numpy()[rows], a)
    assert np.array_equal(out["dist"].cpu().numpy()[rows], dist)
    ctr = out["counters"].cpu().numpy()
    assert ctr[0] + ctr[1] + ctr[2] == n
    return out, so, ctr


@pytest.mark.parametrize("n,d,k", [(255, 64, 66_000), (256, 64, 66_000), (257, 64, 65_600), (2_040, 9, 16_448),
                                   (2_060, 9, 16_400), (1_200, 50, 20_000), (700, 256, 16_384)])
def test_around_the_rule(n, d, k):
    # near-duplicate seeds: nearly every row is left by the bf16 pass
    g = np.random.default_rng(n + d)
    X = (g.uniform(-50, 50, size=(8, d))[g.integers(0, 8, size=n)] + g.normal(size=(n, d))).astype(np.float32)
    sm = g.integers(0, n, size=k).astype(np.uint32)
    out, so, _ = _run(X, sm, np.arange(0, n, max(1, n // 100)), "sizes")
    ref = gpu_api().assign_euclid(cuda(X), cuda(so), cuda(sm), k, 0)
    for name in ("assign", "dist", "sse", "radius"):
        assert torch.equal(out[name], ref[name]), name


@pytest.mark.parametrize("close", [0, 3, 200, 255, 300, 3_000])
def test_few_unsettled_rows(close):
    # seeds far apart but for one pair per `close` row: those rows alone need a rescan
    g = np.random.default_rng(close)
    n, d, k = 6_000, 24, 16_500
    far = g.uniform(-1000, 1000, size=(n, d)).astype(np.float32)
    far[:close] = far[0] + g.normal(size=(close, d)).astype(np.float32) * 1e-3
    sm = (np.arange(k) % n).astype(np.uint32)
    sm[n:] = sm[n] if close == 0 else 0   # the repeated seeds are all one row's
    _, _, ctr = _run(far, sm, np.unique(np.concatenate([np.arange(min(close, 60)), np.arange(0, n, 60)])), "unsettled")
    assert ctr[0] > 0


@pytest.mark.parametrize("n,d,k", [(300, 5, 262_300), (260, 3, 530_000)])
def test_more_groups_than_the_lists_hold(n, d, k):
    g = np.random.default_rng(k)
    X = g.normal(size=(n, d)).astype(np.float32)
    sm = g.integers(0, n, size=k).astype(np.uint32)
    _run(X, sm, np.arange(0, n, 7), "groups")


def test_device_seed_count_batch_and_graph():
    # the same seeds as a host count, as a device count with capacity to spare,
    # in a batched call, and recorded in a graph whose rows change between replays
    api = gpu_api()
    g = np.random.default_rng(9)
    n, d, k, cap = 2_100, 40, 16_500, 16_700
    centers = g.uniform(-50, 50, size=(8, d))
    sets = [torch.from_numpy((centers[g.integers(0, 8, size=n)] + g.normal(size=(n, d)) * s).astype(np.float32)).cuda()
            for s in (1.0, 3.0, 0.01)]
    sm = cuda(g.integers(0, n, size=cap).astype(np.uint32))
    so = torch.arange(cap + 1, dtype=torch.int32, device="cuda")
    kd = torch.tensor([k], dtype=torch.int32, device="cuda")
    announce(f"assign blocked graph n={n} d={d} k={k}")

    def plain(X):
        return api.assign_euclid(X, so[:k + 1], sm[:k], k, 1)

    def same(a, b):
        for name in ("assign", "dist", "sse", "counters"):
            assert torch.equal(a[name], b[name]), name

    X = sets[0].clone()
    ref = plain(X)
    assert int(ref["counters"][1] + ref["counters"][2]) > 1_000
    same(ref, api.assign_euclid(X, so, sm, cap, 1, k_dev=kd))
    outs, _ = api.assign_euclid_batch([(X, so[:k + 1], sm[:k], k), (X, so[:11], sm[:10], 10)], 1)
    for name in ("assign", "dist", "sse", "radius"):
        assert torch.equal(ref[name], outs[0][name]), name

    status = api.new_status("cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        api.assign_euclid(X, so, sm, cap, 1, k_dev=kd, status=status, check=False)  # grows the stream's workspace
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        rec = api.assign_euclid(X, so, sm, cap, 1, k_dev=kd, status=status, check=False)
    for Y in sets[1:] + sets[:1]:
        X.copy_(Y)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        same(plain(X), rec)
