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
