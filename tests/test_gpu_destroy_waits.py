"""A table is destroyed once the work queued for it has run, on whatever stream the latest call queued it: a sorted
export and a migration still read the table when they return."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


def _filled(dev, n, dim):
    from paper_2209_07663_amd.binding import Table
    tab = Table(1 << 22, dim, 5, max_ids=n, device=dev)
    tab.mono_lookup_or_insert(torch.arange(n, device=dev), 0)
    torch.cuda.synchronize()
    return tab


def test_destroy_waits_for_a_sorted_export_on_another_stream():
    from paper_2209_07663_amd.binding import check, device_pointer as p
    dev, n, dim = torch.device("cuda:0"), 2000000, 128
    tab = _filled(dev, n, dim)
    arena = tab.arena                                                   # (kept, so that a failure reads nothing freed)
    keys, row = torch.empty(n, dtype=torch.int64, device=dev), torch.empty(n, dtype=torch.int32, device=dev)
    values = torch.empty((n, dim), device=dev)
    work = torch.empty(tab.lib.mono_export_sorted_bytes(n), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    side, got = torch.cuda.Stream(device=dev), ctypes.c_uint64()
    check(tab.lib.mono_export_sorted(tab.h, 0, p(keys), p(row), None, None, p(values), None, n, p(work), work.numel(),
                                     ctypes.byref(got), side.cuda_stream), "mono_export_sorted")
    tab.close()
    assert side.query() and got.value == n and arena is not None


def test_destroy_of_the_source_waits_for_a_migration_on_another_stream():
    dev, n, dim = torch.device("cuda:0"), 2000000, 128
    src = _filled(dev, n, dim)
    arena, side = src.arena, torch.cuda.Stream(device=dev)
    with torch.cuda.stream(side):
        dst = src.rehashed(1 << 23, 1)
    src.close()
    assert side.query() and arena is not None
    assert dst.mono_table_stats()["size"] == n
    dst.close()
