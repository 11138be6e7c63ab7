"""gather_pool where its work split changes: bags around multiples of the indices a lane holds, empty and very
long bags, numbers of bags around the sizes at which a wave owns fewer of them, rows that fill a lane group,
do not, and are wider than a wave; against a plain fp64 sum over the table's own rows."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EDGE_LENGTHS = [0, 1, 2, 7, 8, 9, 15, 16, 17, 0, 33, 1000]


def _dense_rows(tab):
    d = tab.mono_table_export()
    e = np.zeros((tab.capacity, tab.dim))
    e[d["row"]] = d["rows"]
    return e


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dim", [4, 20, 36, 64, 256, 512, 768, 1024])
def test_pooled_rows_at_the_edges_of_the_work_split(dim, bf16):
    from paper_2209_07663_amd.binding import Table
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(dim + bf16)
    tab = Table(1 << 12, dim, 3, bf16=bf16, max_ids=1 << 20, max_bags=1 << 19, device=dev)
    tab.mono_lookup_or_insert(torch.arange(3000, dtype=torch.int64, device=dev), 0)
    e = _dense_rows(tab)
    bag_counts = [1, 3, 64, 65, 1000] if dim > 64 else [1, 63, 4096 * 8 + 5, 4096 * 64 + 1]
    for bags in bag_counts:
        for lengths in ([np.resize(EDGE_LENGTHS, bags)] if bags <= 1000 else []) + [rng.integers(0, 3, bags)]:
            offsets = np.zeros(bags + 1, dtype=np.int64)
            np.cumsum(lengths, out=offsets[1:])
            n = int(offsets[-1])
            rows = rng.integers(-1, 3000, n).astype(np.int32)
            got = tab.mono_gather_pool(torch.from_numpy(rows).to(dev), torch.from_numpy(offsets).to(dev)).cpu().numpy()
            ref = np.zeros((bags, dim))
            picked = e[np.maximum(rows, 0)] * (rows >= 0)[:, None]
            full = lengths > 0
            if full.any():
                ref[full] = np.add.reduceat(picked, offsets[:-1][full], axis=0)
            scale = np.abs(ref).max(axis=1, keepdims=True) + 1e-30
            assert (np.abs(got - ref) <= 2e-6 * np.sqrt(lengths + 1)[:, None] * np.maximum(scale, 0.0625)).all(), (bags, dim)
    tab.close()
