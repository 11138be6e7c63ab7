"""Which calls of tables without expiry look at a key's counters before its buckets: the ones after a call in which enough
keys missed, whether their counters kept them out or (large batches) they were new and admitted at once.  The device
keeps the answer in its control block, which the test reads from the table's arena; presence, rows and counters are the
oracle's whichever way the next call takes."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu

COUNTERS_FIRST = 64 + 8 * 12      # byte of the control block: four 32-bit and six 64-bit counters, then scratch words


def _counters_first(tab):
    up = lambda v: (v + 255) & ~255
    at = sum(up(v) for v in (16 * tab.capacity, 8 * tab.n_filter, 4 * tab.dim * tab.capacity, 8 * tab.capacity,
                             4 * tab.capacity)) + COUNTERS_FIRST
    return int(tab.arena[at:at + 8].cpu().numpy().view(np.uint64)[0])


@pytest.mark.parametrize("n,threshold,share,want", [
    (70000, 3, 0.02, 0), (70000, 3, 0.2, 1), (70000, 1, 1.0, 0), (70000, 0, 0.5, 0),
    (1 << 19, 3, 0.2, 1), (1 << 19, 1, 1.0, 0),
    ((1 << 19) + 1, 3, 0.1, 0), ((1 << 19) + 1, 3, 0.15, 1), ((1 << 19) + 1, 1, 0.1, 0), ((1 << 19) + 1, 1, 0.15, 1),
    ((1 << 19) + 1, 0, 1.0, 1)])
def test_order_of_the_next_call_follows_the_misses_of_this_one(n, threshold, share, want):
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap, dim = torch.device("cuda:0"), 11, 1 << 22, 4
    rng = np.random.default_rng(n + threshold)
    tab = Table(cap, dim, seed, threshold, 0, max_ids=1 << 20, device=dev, filter_log2=22)
    orc = Oracle(cap, dim, seed, threshold, 0, False, kind="map", n_filter=tab.n_filter)
    known = rng.integers(0, 1 << 40, 50000).astype(np.int64)

    def lookup(keys, step):
        rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step).cpu().numpy()
        assert np.array_equal(rows >= 0, orc.lookup_or_insert(keys, step))

    for _ in range(max(threshold, 1)):
        lookup(known, 0)
    for step in (1, 2):                                       # the second one in the order that the first one asked for
        keys = known[rng.integers(0, known.shape[0], n)]
        absent = rng.random(n) < share
        keys[absent] = rng.integers(1 << 41, 1 << 60, int(absent.sum()))
        lookup(keys, step)
        assert _counters_first(tab) == want
    lookup(known[rng.integers(0, known.shape[0], n)], 3)      # and back
    assert _counters_first(tab) == 0
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=True)
    assert (tab.mono_filter_export() == orc.filter_words()).all()
    tab.close()
