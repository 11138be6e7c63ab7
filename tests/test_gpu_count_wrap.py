"""Occurrence counts are kept in 32 bits and read as at most 255.  On a table without expiry nothing but the host keeps
track of how much a counter can have taken: a key that is turned away for as long as the table is full is counted
2^32 times and more here, and neither its count nor the stored keys that share its counters may suffer."""
import pytest
import torch

from tests import table_checks as tc

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("hashes", [1, 2])
def test_a_count_never_wraps(hashes):
    from paper_2209_07663_amd.binding import Table
    dev, seed, n = torch.device("cuda:0"), 5, 1 << 24
    tab = Table(16, 4, seed, 1, 0, max_ids=n, max_bags=16, device=dev, filter_hashes=hashes, filter_log2=4)
    stored = torch.arange(16, device=dev) * 7919 + 1
    assert (tab.mono_lookup_or_insert(stored, 0) >= 0).all()
    absent = torch.full((n,), 104729, dtype=torch.int64, device=dev)
    counters = [int(tc.filter_index([104729], 16, seed, j)[0]) for j in range(hashes)]
    rows = torch.empty(n, dtype=torch.int32, device=dev)
    for call in range(1, 260):                                    # 2^32 occurrences after 256 calls
        tab.mono_lookup_or_insert(absent, call, rows)
        if call in (1, 2) or call > 120:
            counts = tab.mono_filter_export() & 0xFF
            assert all(counts[c] == 255 for c in counters), call
    assert (rows == -1).all() and tab.mono_table_stats()["n_full"] == 259
    found = tab.mono_lookup_or_insert(stored, 260)                # by the one-kernel lookup
    assert (found >= 0).all()
    mixed = absent.clone()
    mixed[:: n // 1024] = stored[0]                               # and by the general one, which asks the counters first
    tab.mono_lookup_or_insert(mixed, 261, rows)
    assert (rows[:: n // 1024] == found[0]).all() and int((rows >= 0).sum()) == 1024
    tab.close()
