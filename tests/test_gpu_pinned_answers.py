"""Deltas that a program keeps stop taking pinned memory at the allowance, and start again once it lets go of them."""
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_kept_exports_do_not_pin_the_host_without_bound(monkeypatch):
    from paper_2209_07663_amd import binding
    gc.collect()
    monkeypatch.setattr(binding, "PINNED_HELD", binding._pinned.held + (3 << 20), raising=True)
    dev, n, dim = torch.device("cuda:0"), 8192, 16
    tab = binding.Table(1 << 16, dim, 5, max_ids=n, device=dev)
    tab.mono_lookup_or_insert(torch.arange(n, device=dev), 0)
    pinned = lambda d: torch.from_numpy(d["rows"]).is_pinned()
    kept = [tab.mono_table_export() for _ in range(8)]          # 512 KB of rows each, and 230 KB of the rest
    assert pinned(kept[0]) and not pinned(kept[-1]) and sum(map(pinned, kept)) in (3, 4)
    for d in kept[1:]:
        for name in d:
            assert (d[name] == kept[0][name]).all()
    kept.clear()
    gc.collect()
    assert pinned(tab.mono_table_export())
    tab.close()
