"""Host-side check of geek_silk_seeds' workspace: the SILK tables processed
together stay within what a launch holds and what their entries take, however
many tables a small job has."""

import pytest

from paper_2106_10515_amd import _lib as L


def _workspace(n, T, tables):
    return L.workspace_size(L.GEEK_OP_SILK, [L.SilkJob(n=n, T=T, K=1, members=16, offsets=16, nbuckets=16, L=tables,
                                                       delta=2, silk_keys=16, cap_k=8, cap_members=64, seed_offsets=16,
                                                       seed_members=16, k_out=16, needed=16)])


@pytest.mark.parametrize("n,T", [(1, 1), (6, 3), (100, 5)])
def test_many_tables_of_few_entries(n, T):
    # 2^23 entries of 512 at least: 16,384 tables, each with 4 KB of slots
    assert _workspace(n, T, 2_000_000) == _workspace(n, T, 16_384)
    assert _workspace(n, T, 16_384) < 16_384 * (4096 + 100 * n * T) + (1 << 20)
