"""The sweep looks only at buckets whose noted bound of last-seen steps says that a key may be too old.  Streams whose
keys stay, fade and come back, for expiry times below, at and above the largest that is kept to the step, with
sweeps at every step, at random ones and so far apart that bounds no longer say anything; on sparse tables, on
tables full enough for evictions, with restored keys of any age, with and without the list of removed keys;
bit for bit against the oracle at every sweep."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


def _sweep(tab, orc, now, listed, dev):
    n_exp = torch.zeros(1, dtype=torch.int64, device=dev)
    out = torch.full((tab.capacity,), -1, dtype=torch.int64, device=dev) if listed else None
    tab.mono_expire_sweep(now, n_exp, out)
    want = orc.expire_sweep(now)
    n = int(n_exp.item())
    assert n == want.shape[0], "step %d: %d removed, %d expected" % (now, n, want.shape[0])
    if listed:
        assert (np.sort(out[:n].cpu().numpy()) == np.sort(want.astype(np.int64))).all()
    return n


@pytest.mark.parametrize("capacity,per_step", [(16, 2), (1 << 12, 60), (1 << 12, 330), (1 << 19, 3000)])
@pytest.mark.parametrize("expire,gap", [(1, 1), (3, 1), (7, 3), (100, 13), (101, 40), (250, 30), (1000, 90), (60, 400)])
def test_sweeps_remove_what_the_oracle_removes(capacity, per_step, expire, gap):
    """Steps advance by about expire / 7 (or by `gap` with sweeps that far apart)."""
    from paper_2209_07663_amd.binding import Table
    dev, seed = torch.device("cuda:0"), 31
    rng = np.random.default_rng(expire * 7 + capacity)
    tab = Table(capacity, 4, seed, 1, expire, max_ids=8192, device=dev)
    orc = Oracle(capacity, 4, seed, 1, expire, False, kind="cuckoo")
    keys_all = rng.integers(0, 1 << 62, 40 * per_step).astype(np.int64)
    step, removed = 5, 0
    for turn in range(40):
        mine = keys_all[(turn // 2) * per_step:(turn // 2 + 1) * per_step]          # this turn's, last turn's or new ones
        old = keys_all[rng.integers(0, (turn // 2 + 1) * per_step, max(1, per_step // 4))]  # and some of any age
        keys = np.concatenate([mine, old])
        tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step)
        orc.lookup_or_insert(keys, step)
        if gap == 1 or turn % 3 == 2:
            removed += _sweep(tab, orc, step, turn % 2 == 0, dev)
        step += int(rng.integers(1, max(2, expire // 4))) if gap < 100 else int(rng.integers(1, gap))
    removed += _sweep(tab, orc, step, True, dev)
    d = tab.mono_table_export()
    tc.assert_same_table(d, orc.dump(), exact_rows=True)
    removed += _sweep(tab, orc, step + expire, False, dev)                         # everything goes
    assert removed > 0 and tab.mono_table_stats()["size"] == 0 and tab.mono_table_stats()["n_lost"] == 0
    keys = keys_all[:per_step]
    tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step + expire)        # and comes back to emptied buckets
    orc.lookup_or_insert(keys, step + expire)
    assert _sweep(tab, orc, step + expire, True, dev) == 0
    assert _sweep(tab, orc, step + 2 * expire, True, dev) == np.unique(keys).shape[0] or capacity == 16
    tab.close()


@pytest.mark.parametrize("capacity", [1 << 12, 1 << 26])
def test_restored_and_migrated_keys_of_any_age_expire_in_time(capacity):
    from paper_2209_07663_amd.binding import Table
    dev, seed, expire, n = torch.device("cuda:0"), 37, 20, 3000
    rng = np.random.default_rng(capacity)
    tab = Table(capacity, 4, seed, 1, expire, max_ids=8192, device=dev, filter_log2=16)
    orc = Oracle(capacity, 4, seed, 1, expire, False, kind="cuckoo", n_filter=1 << 16)
    keys = np.unique(rng.integers(0, 1 << 62, n + 10).astype(np.int64))[:n]
    seen = rng.integers(0, 1000, n).astype(np.uint32)
    rows, acc = rng.standard_normal((n, 4)).astype(np.float32), rng.random(n).astype(np.float32)
    assert tab.mono_table_import(torch.from_numpy(keys).to(dev), torch.from_numpy(rows).to(dev), torch.from_numpy(acc).to(dev),
                                 torch.from_numpy(seen.view(np.int32)).to(dev)) == 0
    orc.import_entries(keys, rows, acc, seen)
    tables = [(tab, orc)]
    if capacity == 1 << 12:
        grown = tab.rehashed(2 * capacity, 1)
        orc2 = Oracle(capacity, 4, seed, 1, expire, False, kind="cuckoo", n_filter=1 << 16)
        orc2.import_entries(keys, rows, acc, seen)
        orc2.rehash(2 * capacity, 1)
        tables.append((grown, orc2))
    for t, o in tables:
        left = n
        for now in (1000, 1001, 1003, 1007, 1008, 1015, 1018, 1019):
            left -= _sweep(t, o, now, now % 2 == 0, dev)
        assert left == 0
        t.close()
