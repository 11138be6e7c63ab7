"""Tables on either side of the sizes from which a sweep takes two kernels and from which its waves take several shares of the
buckets: keys all over the table, expire, stay or come back; every sweep removes the oracle's keys."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2,expire", [(23, 3), (23, 205), (24, 3), (27, 3), (28, 3), (28, 205)])
def test_sweeps_remove_what_the_oracle_removes(log2, expire):
    from paper_2209_07663_amd.binding import Table
    dev, seed = torch.device("cuda:0"), 41
    rng = np.random.default_rng(log2 + expire)
    tab = Table(1 << log2, 4, seed, 1, expire, max_ids=1 << 17, device=dev, filter_log2=16)
    orc = Oracle(1 << 20, 4, seed, 1, expire, False, kind="map", n_filter=1 << 16)
    keys_all = rng.integers(0, 1 << 62, 300000).astype(np.int64)
    step, removed, count = 3, 0, torch.zeros(1, dtype=torch.int64, device=dev)
    for turn in range(8):
        keys = np.concatenate([keys_all[turn * 30000:turn * 30000 + 40000], keys_all[rng.integers(0, 300000, 3000)]])
        tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step)
        orc.lookup_or_insert(keys, step)
        out = torch.full((1 << 18,), -1, dtype=torch.int64, device=dev) if turn % 2 else None
        tab.mono_expire_sweep(step, count, out)
        want = np.sort(orc.expire_sweep(step).astype(np.int64))
        assert int(count.item()) == want.shape[0]
        if out is not None:
            assert (np.sort(out[:want.shape[0]].cpu().numpy()) == want).all()
        removed += want.shape[0]
        step += max(1, expire // 3)
    assert removed > 0
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=True)
    tab.close()
