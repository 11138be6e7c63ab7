"""Small batches go through a lookup kernel of their own: the sizes at its edges (one key, a block's 256 keys, the
largest batch it takes and the smallest it leaves to the general path), all-hit, all-miss and mixed batches with
duplicates and padding, every kind of counter, and a table driven through evictions to its fill limit; bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 255, 256, 257, 1500, 4095, 4096, 4097]


def _check(tab, orc, keys, step, dev):
    rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step).cpu().numpy()
    present = orc.lookup_or_insert(keys, step)
    assert ((rows >= 0) == present).all() and (rows >= -1).all(), "step %d" % step
    d = tab.mono_table_export()
    tc.assert_same_table(d, orc.dump(), exact_rows=True)
    tc.check_placement(d, tab.capacity, 8, tab.seed)
    row_of = dict(zip(d["keys"].tolist(), d["row"].tolist()))
    assert all(r == row_of[k] for k, r in zip(keys.tolist(), rows.tolist()) if r >= 0), "a key resolved to another row"
    assert (tab.mono_filter_export() == orc.filter_words()).all(), "counter words differ at step %d" % step


@pytest.mark.parametrize("threshold,expire,hashes,bf16,dim", [(1, 0, 1, False, 16), (3, 0, 2, True, 8), (2, 3, 1, False, 36),
                                                               (0, 2, 3, False, 4), (255, 0, 1, False, 4)])
def test_small_batches_match_the_oracle(threshold, expire, hashes, bf16, dim):
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap = torch.device("cuda:0"), 7 + threshold, 1 << 15
    rng = np.random.default_rng(seed)
    tab = Table(cap, dim, seed, threshold, expire, bf16, max_ids=8192, device=dev, filter_hashes=hashes)
    orc = Oracle(cap, dim, seed, threshold, expire, bf16, kind="cuckoo", n_filter=tab.n_filter, filter_hashes=hashes)
    step = 0
    for n in SIZES + SIZES[::-1]:
        fresh = rng.integers(0, 1 << 62, n)                             # hardly a key twice
        pool = rng.integers(0, 3000, n)                                 # keys of earlier batches, many of them twice
        keys = np.where(rng.random(n) < rng.choice([0.0, 0.2, 0.9]), fresh, pool).astype(np.int64)
        keys[rng.random(n) < 0.02] = -1
        for k in (keys, keys):                                          # the second time most of it is known
            _check(tab, orc, k, step, dev)
            step += 1
        if expire:
            n_exp = torch.zeros(1, dtype=torch.int64, device=dev)
            tab.mono_expire_sweep(step, n_exp)
            assert int(n_exp.item()) == orc.expire_sweep(step).shape[0]
    st = tab.mono_table_stats()
    assert st["n_lost"] == 0 and st["n_insert_failed"] == 0
    tab.close()


def test_small_batches_fill_a_table_to_its_limit_and_are_refused_whole():
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap = torch.device("cuda:0"), 23, 1 << 12
    rng = np.random.default_rng(seed)
    tab = Table(cap, 4, seed, 1, 4, False, max_ids=4096, device=dev)
    orc = Oracle(cap, 4, seed, 1, 4, False, kind="cuckoo")
    for step in range(16):
        _check(tab, orc, rng.integers(0, 1 << 62, 700).astype(np.int64), step, dev)
        assert tab.mono_table_stats()["n_full"] == orc.refused_full
        if step % 8 == 7:
            n_exp = torch.zeros(1, dtype=torch.int64, device=dev)
            tab.mono_expire_sweep(step, n_exp)
            assert int(n_exp.item()) == orc.expire_sweep(step).shape[0] > 0
    st = tab.mono_table_stats()
    assert st["n_lost"] == 0 and st["n_full"] > 0
    tab.close()
