"""Lookups whose step lies behind the latest sweep (accepted: only lookups are held to non-decreasing steps).  They
stamp stored keys with, and bring new ones at, steps that are older than the bounds which the sweep has noted for their
buckets: the next sweep must find them all the same.  By the one-kernel lookup and by the general path, on tables
small and large enough for either width of the sweep; against the oracle at every sweep."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc
from tests.test_gpu_sweep_bounds import _sweep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("capacity", [1 << 16, 1 << 26])
@pytest.mark.parametrize("expire", [20, 1000])
@pytest.mark.parametrize("n", [300, 6000])
def test_keys_of_a_lookup_behind_the_sweep_expire_in_time(n, expire, capacity):
    from paper_2209_07663_amd.binding import Table
    dev, seed, top = torch.device("cuda:0"), 41, 100 * expire
    rng = np.random.default_rng(n + expire)
    tab = Table(capacity, 4, seed, 1, expire, max_ids=1 << 15, device=dev, filter_log2=16)
    orc = Oracle(1 << 16, 4, seed, 1, expire, False, kind="map", n_filter=1 << 16)
    keys = np.unique(rng.integers(0, 1 << 62, 3 * n + 10).astype(np.int64))
    old, new, later = rng.permutation(keys)[:3 * n].reshape(3, n)
    seen = (top - 1 - rng.integers(0, expire // 4, n)).astype(np.uint32)
    rows, acc = rng.standard_normal((n, 4)).astype(np.float32), rng.random(n).astype(np.float32)
    assert tab.mono_table_import(torch.from_numpy(old).to(dev), torch.from_numpy(rows).to(dev),
                                 torch.from_numpy(acc).to(dev), torch.from_numpy(seen.view(np.int32)).to(dev)) == 0
    orc.import_entries(old, rows, acc, seen)

    def lookup(k, step):
        got = tab.mono_lookup_or_insert(torch.from_numpy(k).to(dev), step).cpu().numpy()
        assert ((got >= 0) == orc.lookup_or_insert(k, step)).all()

    assert _sweep(tab, orc, top, False, dev) == 0                                  # notes the bounds of the old keys
    lookup(np.concatenate([old[:n // 2], new]), top // 2)                          # far behind it
    assert _sweep(tab, orc, top + expire // 2, True, dev) == n // 2 + n            # all that the lookup saw goes
    lookup(np.concatenate([old[n // 2: 3 * n // 4], new]), top + expire // 4)      # a little behind it
    for now in (top + expire // 2, top + expire, top + expire + expire // 4 - 1, top + expire + expire // 4):
        _sweep(tab, orc, now, now % 2 == 0, dev)
    lookup(later, top + 2 * expire)
    assert _sweep(tab, orc, top + 3 * expire - 1, True, dev) == 0
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=True)
    assert _sweep(tab, orc, top + 3 * expire, False, dev) == n and tab.mono_table_stats()["size"] == 0
    tab.close()
