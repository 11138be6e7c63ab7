"""How the update groups its pairs follows from the size of the batch (one block in LDS up to 4096 pairs, the split up to 2^20,
radix passes beyond) and, of the radix passes, from the rows in use (8- or 9-bit digits): batches at the edges of each, with
hot rows, dropped occurrences and bags of every length, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from tests import table_checks as tc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 1025, 4095, 4096, 4097, 8191, 8192, 8193, 50001, 400000, 400001, 1 << 20, (1 << 20) + 1])
def test_update_at_the_edges_of_the_sort_shapes(n):
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap, dim = torch.device("cuda:0"), 11, 1 << 18, 8
    rng = np.random.default_rng(n)
    tab = Table(cap, dim, seed, 1, 0, max_ids=1 << 21, max_bags=1 << 21, device=dev)
    orc = Oracle(cap, dim, seed, 1, 0, False, kind="cuckoo")
    known = rng.permutation(np.unique(rng.integers(0, 1 << 40, 210000)))[:200000].astype(np.int64)
    tab.mono_lookup_or_insert(torch.from_numpy(known).to(dev), 0)
    orc.lookup_or_insert(known, 0)
    for step, empty in ((1, False), (2, True)):                       # the second time with many empty bags
        keys = known[np.minimum(rng.zipf(1.2, n) - 1, 199999)]
        spread = rng.random(n) < 0.5
        keys[spread] = known[rng.integers(0, 200000, int(spread.sum()))]
        keys[rng.random(n) < 0.05] = -1
        lengths = rng.poisson(3.0, n + 1) * (rng.random(n + 1) < (0.3 if empty else 1.0))
        offs = np.concatenate([[0], np.minimum(np.cumsum(lengths), n)]).astype(np.int64)
        offs[-1] = n
        if empty:
            offs = np.concatenate([offs, np.full(20000, n)]).astype(np.int64)
        grad = rng.standard_normal((offs.shape[0] - 1, dim)).astype(np.float32)
        rows = tab.mono_lookup_or_insert(torch.from_numpy(keys).to(dev), step)
        orc.lookup_or_insert(keys, step)
        tab.mono_apply_grad_adagrad(rows, torch.from_numpy(offs).to(dev), torch.from_numpy(grad).to(dev), 0.05, 1e-6)
        orc.apply_grad_adagrad(keys, offs, grad, 0.05, 1e-6)
    tc.assert_same_table(tab.mono_table_export(), orc.dump(), exact_rows=False, rtol=2e-5)
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()


@pytest.mark.parametrize("n", [3000, 9000, (1 << 20) + 5])
def test_wide_digits_in_small_and_large_batches(n):
    """More than 2^24 rows in use: two batches of 9 M new keys raise the mark, then an update is compared that one block sorts
    (in four digits), one that is split and one of nine-bit digits."""
    from paper_2209_07663_amd.binding import Table
    dev, seed, cap, dim = torch.device("cuda:0"), 13, 1 << 25, 4
    tab = Table(cap, dim, seed, 1, 0, max_ids=9 << 20, max_bags=9 << 20, device=dev)
    for step in range(2):
        tab.mono_lookup_or_insert(torch.arange(9 << 20, device=dev) + step * (9 << 20), step)
    rng = np.random.default_rng(n)
    keys = torch.from_numpy(np.where(rng.random(n) < 0.3, rng.integers(0, 50, n), rng.integers(0, 18 << 20, n))).to(dev)
    rows = tab.mono_lookup_or_insert(keys, 2)
    assert int(rows.max()) >= 1 << 24
    offs = torch.arange(n + 1, device=dev)
    before = tab.mono_gather_pool(rows, offs)
    grad = torch.from_numpy(rng.standard_normal((n, dim)).astype(np.float32)).to(dev)
    tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
    after = tab.mono_gather_pool(rows, offs).double().cpu().numpy()
    r, first, inv = np.unique(rows.cpu().numpy(), return_index=True, return_inverse=True)
    g = np.zeros((r.shape[0], dim))
    np.add.at(g, inv, grad.double().cpu().numpy())
    acc = (g * g).mean(axis=1, keepdims=True)
    want = before.double().cpu().numpy()[first] - 0.05 * g / (np.sqrt(acc) + 1e-6)
    tc.rows_close(after[first], want, 1e-5)
    tab.close()
