"""Large batches: pooled results of more than 192 MB are stored, and rows of updates of more than 256 MB read and
written, past the caches.  Both sides of each line, against small calls (gather) and a fp64 reduction (update)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dim,n", [(64, (1 << 18) + 1), (64, 786432), (64, 786433), (1024, 65536), (1024, 65537), (1024, 131073), (36, 3728271)])
def test_large_gathers_and_updates(dim, n, bf16):
    from paper_2209_07663_amd.binding import Table
    dev, known = torch.device("cuda:0"), 30000
    g = torch.Generator(device=dev).manual_seed(n)
    tab = Table(1 << 16, dim, 5, bf16=bf16, max_ids=n, max_bags=n, device=dev)
    keys = torch.randint(0, known, (n,), device=dev, generator=g)
    keys[: n // 4] = 7                                          # a hot row of many tiles
    rows = tab.mono_lookup_or_insert(keys, 0)
    each = torch.arange(n + 1, device=dev)
    all_keys = torch.arange(known, device=dev)
    all_rows = tab.mono_lookup_or_insert(all_keys, 0)
    before = tab.mono_gather_pool(all_rows, each[: known + 1])  # a row per key
    assert torch.equal(tab.mono_gather_pool(rows, each), before[keys])
    bags = (n + 2) // 3
    offs = torch.clamp(torch.arange(bags + 1, device=dev) * 3, max=n)
    grad = torch.randn(bags, dim, device=dev, generator=g)
    tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
    after = tab.mono_gather_pool(all_rows, each[: known + 1])
    total = torch.zeros(known, dim, dtype=torch.float64, device=dev)
    for lo in range(0, n, 1 << 18):                             # (in parts: a batch of fp64 gradients is large)
        at = torch.arange(lo, min(lo + (1 << 18), n), device=dev)
        hot = keys[at] == 7                                     # (summed apart: index_add_ is slow where one row repeats)
        total.index_add_(0, keys[at[~hot]], grad[at[~hot] // 3].double())
        total[7] += grad[at[hot] // 3].double().sum(dim=0)
    acc = total.pow(2).mean(dim=1, keepdim=True)
    ref = before.double() - 0.05 * total / (acc.sqrt() + 1e-6)
    tol = 2.0 ** -8 * ref.abs() + 1e-5 if bf16 else 2e-5 * (ref.abs() + 0.05)
    assert ((after.double() - ref).abs() <= tol).all()
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()
