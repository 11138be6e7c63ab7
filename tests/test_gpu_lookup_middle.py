"""Batches between the one-kernel lookup and the large path: the sizes on either side of where both buckets are asked for at
once and where the insertion stops resolving duplicates, new keys that occur once and many times, padding, counters that
age and that do not, and a batch that is refused whole.  Everything is the oracle's, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4097, 5000, 65535, 65536, 65537, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("threshold,expire,hashes", [(1, 0, 1), (3, 0, 2), (2, 3, 1), (3, 2, 3)])
def test_middle_batches_match_the_oracle(n, threshold, expire, hashes):
    from paper_2209_07663_amd.binding import Table
    dev, seed = torch.device("cuda:0"), n + threshold
    cap = 1 << (n // 2).bit_length()                                    # a batch of 1.2 n new keys is more than there is room for
    rng = np.random.default_rng(seed)
    tab = Table(cap, 4, seed, threshold, expire, False, max_ids=n, device=dev, filter_hashes=hashes)
    orc = Oracle(cap, 4, seed, threshold, expire, False, kind="map", n_filter=tab.n_filter, filter_hashes=hashes)
    every = rng.permutation(np.unique(rng.integers(0, 1 << 62, 4 * n))).astype(np.int64)
    few, many = every[: n // 4], every[n // 4:]
    refused = 0
    for step, keys in enumerate([
            few[rng.integers(0, few.size, n)],                          # every key four times
            few[(few.size * rng.random(n) ** 6).astype(np.int64)],      # some hundreds of times
            np.concatenate([few[: n // 2], many[: n - few[: n // 2].size]]),
            many[:n], many[:n], many[:n]]):                             # at a threshold of three the last is refused or admitted
        keys = rng.permutation(keys)
        keys[rng.random(n) < 0.01] = -1
        rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step).cpu().numpy()
        present = orc.lookup_or_insert(keys, step)
        assert ((rows >= 0) == present).all() and (rows >= -1).all(), "step %d" % step
        d = tab.mono_table_export()
        tc.assert_same_table(d, orc.dump(), exact_rows=True)
        tc.check_placement(d, tab.capacity, 8, tab.seed)
        at = np.searchsorted(d["keys"].view(np.uint64), keys[present].view(np.uint64))
        assert np.array_equal(d["row"][at], rows[present]), "a key resolved to another row"
        assert (tab.mono_filter_export() == orc.filter_words()).all(), "counter words differ at step %d" % step
        assert tab.mono_table_stats()["n_full"] == orc.refused_full
        refused = orc.refused_full
        if expire:
            n_exp = torch.zeros(1, dtype=torch.int64, device=dev)
            tab.mono_expire_sweep(step, n_exp)
            assert int(n_exp.item()) == orc.expire_sweep(step).shape[0]
    assert refused > 0
    st = tab.mono_table_stats()
    assert st["n_lost"] == 0 and st["n_insert_failed"] == 0
    tab.close()
