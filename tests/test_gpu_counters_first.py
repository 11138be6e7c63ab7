"""lookup_or_insert on tables without expiry looks at a key's counters before its buckets, or not, by what the call before
saw: batches of known keys, of keys that their counters keep out, and of both, in turn, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threshold,hashes", [(1, 1), (3, 1), (3, 2)])
@pytest.mark.parametrize("n", [5001, 70000, (1 << 19) + 1])
def test_rows_and_counts_whatever_the_call_before_saw(n, threshold, hashes):
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap, dim = torch.device("cuda:0"), 11, 1 << 18, 4
    rng = np.random.default_rng(n + threshold)
    tab = Table(cap, dim, seed, threshold, 0, max_ids=1 << 20, device=dev, filter_hashes=hashes, filter_log2=22)
    orc = Oracle(cap, dim, seed, threshold, 0, False, kind="cuckoo", n_filter=tab.n_filter, filter_hashes=hashes)
    known = rng.integers(0, 1 << 40, 50000).astype(np.int64)
    for _ in range(threshold):
        tab.mono_lookup_or_insert(torch.from_numpy(known).to(dev), 0)
        orc.lookup_or_insert(known, 0)
    for step, share in enumerate((0.0, 1.0, 1.0, 0.3, 0.9, 0.0), start=1):
        keys = known[rng.integers(0, known.shape[0], n)]
        absent = rng.random(n) < (share if threshold > 1 else 0.1 * share)
        keys[absent] = rng.integers(1 << 41, 1 << 60, int(absent.sum()))
        rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step).cpu().numpy()
        ref = orc.lookup_or_insert(keys, step)
        assert np.array_equal(rows >= 0, ref)
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=False, rtol=1e-6)
    tab.close()


@pytest.mark.parametrize("n", [65537, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("threshold,hashes,filter_log2", [(2, 1, 12), (3, 2, 19), (40, 1, 18), (4, 3, 22)])
def test_counters_that_share_marks_and_steps_that_come_twice(n, threshold, hashes, filter_log2):
    """Counter words and admissions where a counter was looked at before it is touched: by a batch of the same step, by many
    blocks of one batch, by several keys; fewer counters than marks and more, and marks of earlier calls."""
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap = torch.device("cuda:0"), 17, 1 << 20
    rng = np.random.default_rng(n + threshold)
    tab = Table(cap, 4, seed, threshold, 0, max_ids=n, device=dev, filter_hashes=hashes, filter_log2=filter_log2)
    orc = Oracle(cap, 4, seed, threshold, 0, False, kind="map", n_filter=tab.n_filter, filter_hashes=hashes)
    keys = rng.permutation(np.unique(rng.integers(0, 1 << 62, 2 * n))).astype(np.int64)
    for call, step in enumerate((0, 1, 1, 2, 7, 7)):
        batch = keys[(keys.size * rng.random(n) ** (1, 2, 1, 4, 1, 3)[call]).astype(np.int64)]
        rows = tab.mono_lookup_or_insert(torch.from_numpy(batch).to(dev), step).cpu().numpy()
        assert np.array_equal(rows >= 0, orc.lookup_or_insert(batch, step)), "call %d" % call
        assert (tab.mono_filter_export() == orc.filter_words()).all(), "counter words differ after call %d" % call
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=True)
    assert tab.mono_table_stats()["n_admitted"] > 0
    tab.close()
