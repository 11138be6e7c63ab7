"""How many new keys a wave of the insertion takes at a time follows from their number and the grid: the numbers on either
side of each change, at the narrowest, odd, ordinary and widest rows.  Rows, values and counters are the oracle's."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


# 5000 IDs are 79 blocks: 8 keys a wave up to 79 * 32 = 2528; from 131072 IDs on there are 2048 blocks
@pytest.mark.parametrize("n,new,dim,bf16", [
    (5000, 1, 512, False), (5000, 2528, 128, False), (5000, 2529, 128, True), (5000, 5000, 12, False),
    (300000, 65536, 4, False), (300000, 65537, 4, True), (300000, 131072, 8, False), (300000, 131073, 8, False),
    (300000, 262144, 4, False), (300000, 262145, 4, False), (300000, 300000, 36, True)])
def test_new_rows_are_the_oracles(n, new, dim, bf16):
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap = torch.device("cuda:0"), 5, 1 << 20
    rng = np.random.default_rng(n + new + dim)
    tab = Table(cap, dim, seed, 1, 0, max_ids=n, device=dev, bf16=bf16)
    orc = Oracle(cap, dim, seed, 1, 0, bf16, kind="map", n_filter=tab.n_filter)
    every = np.unique(rng.integers(0, 1 << 60, 2 * n))
    rng.shuffle(every)
    known, fresh = every[:100], every[100:100 + new]
    for step, keys in enumerate((known, np.concatenate([fresh, known[rng.integers(0, 100, n - new)]]), fresh)):
        keys = rng.permutation(keys).astype(np.int64)
        rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step).cpu().numpy()
        assert np.array_equal(rows >= 0, orc.lookup_or_insert(keys, step))
        by_key = keys[np.argsort(keys, kind="stable")], rows[np.argsort(keys, kind="stable")]
        assert (np.diff(by_key[1])[np.diff(by_key[0]) == 0] == 0).all()           # a key has one row
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=True)
    tab.close()
