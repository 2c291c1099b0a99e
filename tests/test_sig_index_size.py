"""Host-side checks of the signature assignment's sizes at seed counts that no
test can run."""

import pytest

from paper_2106_10515_amd import _lib as L


def _workspace(k, F):
    return L.workspace_size(L.GEEK_OP_ASSIGN, [L.AssignJob(
        metric=L.GEEK_METRIC_SIG, n=1, k=k, sig=16, F=F, n_members=k, seed_offsets=16, seed_members=16, assign=16,
        modes=16, sse=16)])


@pytest.mark.timeout(20)
@pytest.mark.parametrize("k", [2**23 + 1, 2**30, 2**30 + 1, 2**31 - 1])
def test_workspace_of_any_seed_count(k):
    assert _workspace(k, 1) > 24 * k


@pytest.mark.parametrize("k,F,slots", [(2**20, 1024, 2**32), (2**21, 1024, 2**32), (2**22 - 1, 1024, 2**32),
                                       (3 * 2**18, 1024, 2**31)])
def test_index_has_room(k, F, slots):
    # more slots than entries, so that every probe ends; 16 bytes a slot, the
    # other arrays take at least six words an entry
    assert slots > k * F and _workspace(k, F) >= slots * 16 + k * F * 24


@pytest.mark.parametrize("k,F", [(2**22, 1024), (2**31 - 1, 1024), (2**31 - 1, 3)])
def test_index_past_32_bits_is_refused(k, F):
    with pytest.raises(L.GeekError, match="unsupported"):
        _workspace(k, F)
