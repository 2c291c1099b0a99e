"""Host-side check of geek_quantile_buckets' workspace: eight bytes a (table,
object) for the values, as many tables as there are, and the records of the
tables ranked together."""

import pytest

from paper_2106_10515_amd import _lib as L


def _workspace(n, m, t):
    return L.workspace_size(L.GEEK_OP_QUANTILE, [L.QuantileJob(n=n, d=8, m=m, t=t, X=16, ldx=8, A=16, members=16,
                                                               offsets=16)])


@pytest.mark.parametrize("n", [100_000, 10_000_000, 24_000_000])
@pytest.mark.parametrize("m", [1, 3, 9])
@pytest.mark.parametrize("t", [10_000, 3])
def test_workspace_of_few_tables(n, m, t):
    # values, then 20 bytes a record of at most 2 GB of tables; a tenth for
    # counts and splitters, which small tables round up
    group = min(m, max(1, (2 << 30) // (20 * n)))
    assert _workspace(n, m, t) < (8 * m + 20 * group) * n * 1.1 + (1 << 20)


def test_workspace_past_the_sample_sort():
    n = 30_000_000
    assert _workspace(n, 1, 10_000) < (8 + 24) * n * 1.05 + (1 << 20)
