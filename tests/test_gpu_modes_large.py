"""GPU parity of the signature assignment's modes with numpy, bit for bit, at
member counts past what one 32-bit sort can hold."""

import numpy as np
import pytest

from .gpu_util import announce, cuda, gpu_api, host_u32

pytestmark = pytest.mark.gpu


def _modes(sig, so, sm, values):
    """Most frequent value per seed and position (the smallest on ties) of
    members that repeat, by counts per object; values lie in 0 .. values - 1."""
    out = []
    for j in range(len(so) - 1):
        times = np.bincount(sm[so[j]:so[j + 1]], minlength=len(sig)).astype(np.float64)
        out.append(np.argmax([times @ (sig == v) for v in range(values)], axis=0))
    return np.array(out, np.uint32)


def test_more_than_2_to_32_items():
    # 64 seeds of 65,700 members and 1,024 positions: 4.3 10^9 items
    api = gpu_api()
    g = np.random.default_rng(0)
    n, F, k, per, values = 500, 1024, 64, 65_700, 5
    sig = g.integers(0, values, size=(n, F)).astype(np.uint32)
    so = (np.arange(k + 1) * per).astype(np.uint32)
    sm = g.integers(0, n, size=k * per).astype(np.uint32)
    assert len(sm) * F > 2**32
    announce(f"modes n={n} F={F} k={k} members={len(sm)}")
    out = api.assign_sig(cuda(sig), cuda(so), cuda(sm), k)
    api.release_workspace()
    modes = _modes(sig, so, sm, values)
    assert np.array_equal(host_u32(out["modes"]), modes)
    match = (sig[:, None, :] == modes[None]).sum(axis=2)
    assert np.array_equal(out["assign"].cpu().numpy(), np.argmax(match, axis=1))


@pytest.mark.parametrize("per,given", [(4, 7), (60, 100), (60, 61)])
def test_seeds_past_the_member_count_are_refused(per, given):
    # seed_offsets that claim more members than the job has ids for
    api = gpu_api()
    g = np.random.default_rng(1)
    n, F, k = 200, 12, 3
    sig, cat = g.integers(0, 9, size=(n, F)).astype(np.uint32), g.integers(0, 9, size=(n, 5)).astype(np.uint32)
    X = g.normal(size=(n, 3)).astype(np.float32)
    so = (np.arange(k + 1) * per).astype(np.uint32)
    sm = g.integers(0, n, size=k * per).astype(np.uint32)
    announce(f"modes past the member count per={per} given={given}")
    whole, ids = cuda(sm), cuda(sm)[:given]
    for call in (lambda m: api.assign_sig(cuda(sig), cuda(so), m, k),
                 lambda m: api.assign_hetero(cuda(X), cuda(cat), cuda(so), m, k, 1.0, 1)):
        with pytest.raises(api.GeekError, match="invalid argument"):
            call(ids)
        call(whole)


def test_more_seeds_than_one_launch_of_workgroups():
    # 2^24 seeds: a workgroup of 256 threads each would be 2^32 threads
    api = gpu_api()
    g = np.random.default_rng(2)
    n, F, k = 40, 2, 2**24 + 3
    sig = g.integers(0, 6, size=(n, F)).astype(np.uint32)
    sm = g.integers(0, n, size=k).astype(np.uint32)
    announce(f"modes n={n} F={F} k={k}")
    out = api.assign_sig(cuda(sig), cuda(np.arange(k + 1, dtype=np.uint32)), cuda(sm), k)
    api.release_workspace()
    assert np.array_equal(host_u32(out["modes"]), sig[sm])
    first = [int(np.flatnonzero((sig[sm[:4000]] == row).all(axis=1))[0]) for row in sig]
    assert out["assign"].cpu().numpy().tolist() == first
