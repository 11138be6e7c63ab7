"""Updates of few pairs, on tables with 2^16 to 2^22 rows in use and one more than that: both sides of what one block sorts, in
pairs and in bags, batches of fewer pairs than the split draws samples, and the split's own smaller sizes; with a hot row, dropped
occurrences and whole units of one row, against an fp64 reduction."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (one block: up to 4096 pairs in up to 16384 bags)
PAIRS_BAGS = [(1, 16385), (60, 40000), (511, 20000), (513, 16385), (4096, 16384), (4096, 16385), (4097, 5000), (8193, 8193),
              (32769, 32769), (65537, 65537), (131073, 131073)]


@pytest.mark.parametrize("used", [65536, 65537, 1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1, 1 << 22, (1 << 22) + 1])
def test_updates_on_both_sides_of_the_lines(used):
    from paper_2209_07663_amd.binding import Table
    dev, dim, most = torch.device("cuda:0"), 4, 1 << 20
    g = torch.Generator(device=dev).manual_seed(used)
    tab = Table(1 << 23, dim, 5, max_ids=most, max_bags=most, device=dev)
    for lo in range(0, used, most):
        tab.mono_lookup_or_insert(torch.arange(lo, min(lo + most, used), device=dev), 0)
    each = torch.arange(most + 1, device=dev)
    acc = torch.zeros(1 << 23, dtype=torch.float64, device=dev)
    for step, (n, bags) in enumerate(PAIRS_BAGS, start=1):
        keys = torch.randint(0, used, (n,), device=dev, generator=g)
        keys[: n // 8] = used - 1                                    # a hot row: whole units of one row
        rows = tab.mono_lookup_or_insert(keys, step)
        rows[n // 2:: 97] = -1
        assert tab.mono_table_stats()["size"] == used                # (the host knows the rows in use exactly now)
        if bags == n:
            offs = each[: n + 1]
        else:
            cut = torch.sort(torch.randint(0, n + 1, (bags - 1,), device=dev, generator=g))[0]
            offs = torch.cat([each[:1], cut, each[n:n + 1]])
        bag = torch.repeat_interleave(each[:bags], offs[1:] - offs[:-1])
        kept = rows >= 0
        at, inv = torch.unique(rows[kept], return_inverse=True)
        before = tab.mono_gather_pool(at, each[: at.numel() + 1]).double()
        grad = torch.randn(bags, dim, device=dev, generator=g)
        tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
        after = tab.mono_gather_pool(at, each[: at.numel() + 1]).double()
        total = torch.zeros(at.numel(), dim, dtype=torch.float64, device=dev)
        per_pair = grad[bag][kept].double()
        if at.numel():
            hot = inv == inv[0]                                      # (summed apart: index_add_ is slow where one row repeats)
            total.index_add_(0, inv[~hot], per_pair[~hot])
            total[inv[0]] += per_pair[hot].sum(dim=0)
        acc[at.long()] += total.pow(2).mean(dim=1)
        ref = before - 0.05 * total / (acc[at.long()].sqrt()[:, None] + 1e-6)
        assert ((after - ref).abs() <= 2e-5 * (ref.abs() + 0.05)).all(), (n, bags)
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()
