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


@pytest.mark.parametrize("n,bags", [(60, 16385), (500, 1 << 20), (4000, 32 * 4000 + 31), (4000, 32 * 4001), (4000, 300000),
                                    (60000, 32 * 60001), (65536, 32 * 65537), (65537, 32 * 65538)])
def test_bags_beyond_those_that_a_unit_walks(n, bags):
    """Occurrences in few of many bags, of the sizes where the split searches bags and of the next ones: on both sides of the
    last bag that the first unit walks over (16 turns of two bags a thread, from bag 0 on here), in the batch's last bag, and
    in bags that span units."""
    from paper_2209_07663_amd.binding import Table
    dev, dim, used, walked = torch.device("cuda:0"), 4, 1 << 16, 8192
    g = torch.Generator(device=dev).manual_seed(n)
    tab = Table(1 << 18, dim, 5, max_ids=1 << 22, max_bags=1 << 22, device=dev)
    tab.mono_lookup_or_insert(torch.arange(used, device=dev), 0)
    acc = torch.zeros(1 << 18, dtype=torch.float64, device=dev)
    edges = torch.tensor([0, walked - 1, walked, walked + 1, 2 * walked, bags - 1], device=dev)
    for few in (True, False):
        bag = torch.randint(0, bags, (n,), device=dev, generator=g)
        if few:
            bag = edges[torch.randint(0, edges.numel(), (n,), device=dev, generator=g)]
        bag[: edges.numel()] = edges
        bag = torch.sort(bag)[0]
        offs = torch.searchsorted(bag, torch.arange(bags + 1, device=dev))
        rows = tab.mono_lookup_or_insert(torch.randint(0, used, (n,), device=dev, generator=g), 1)
        rows[n // 3] = -1
        # whole numbers below 2^24 in every sum: a pair in a wrong bag shows whatever the order of the sums
        grad = torch.randint(-3, 4, (bags, dim), device=dev, generator=g).float()
        kept = rows >= 0
        at = torch.unique(rows[kept])
        one = torch.arange(at.numel() + 1, device=dev)
        before = tab.mono_gather_pool(at, one).double()
        tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
        after = tab.mono_gather_pool(at, one).double()
        total = torch.zeros(1 << 18, dim, dtype=torch.float64, device=dev)
        total.index_add_(0, rows[kept].long(), grad[bag][kept].double())
        acc += total.pow(2).mean(dim=1)
        ref = before - 0.05 * total[at.long()] / (acc[at.long()].sqrt()[:, None] + 1e-6)
        assert ((after - ref).abs() <= 2e-5 * (ref.abs() + 0.05)).all(), few
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()
