"""The sort's large shapes make histograms for groups of four units: batches whose last group is cut anywhere, and with
more groups than threads scan them, against an fp64 reduction."""
import pytest
import torch

pytestmark = pytest.mark.gpu

UNIT = {False: 2048, True: 4096}  # elements of a unit: digits of 8 bits, of 9


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("units,extra", [(514, 0), (514, 1), (515, 2047), (516, 1), (4 * 1024, 0), (4 * 1024, 1)])
def test_update_at_the_edges_of_the_groups(units, extra, wide):
    from paper_2209_07663_amd.binding import Table
    dev, dim, n = torch.device("cuda:0"), 4, units * UNIT[wide] + extra
    known = (9 << 20) * 2 if wide else 300000            # more than 2^24 rows in use: 9-bit digits
    g = torch.Generator(device=dev).manual_seed(n)
    tab = Table(1 << 25 if wide else 1 << 20, dim, 5, max_ids=max(n, 9 << 20), max_bags=n, device=dev)
    for lo in range(0, known, 9 << 20):
        tab.mono_lookup_or_insert(torch.arange(lo, min(lo + (9 << 20), known), device=dev), 0)
    keys = torch.randint(0, known, (n,), device=dev, generator=g)
    keys[: n // 8] = 7                                   # a hot row: whole units of one digit
    rows = tab.mono_lookup_or_insert(keys, 1)
    rows[n // 2 :: 97] = -1                              # dropped occurrences
    each = torch.arange(known + 1, device=dev)
    all_rows = torch.cat([tab.mono_lookup_or_insert(each[lo : min(lo + (9 << 20), known)], 1)
                          for lo in range(0, known, 9 << 20)])
    table_row = torch.empty(1 << 25, dtype=torch.int64, device=dev)
    table_row[all_rows.long()] = each[:-1]

    def values():
        return torch.cat([tab.mono_gather_pool(all_rows[lo : lo + 500000], each[: min(500000, known - lo) + 1])
                          for lo in range(0, known, 500000)])
    before = values()
    bags = (n + 2) // 3
    offs = torch.clamp(torch.arange(bags + 1, device=dev) * 3, max=n)
    grad = torch.randn(bags, dim, device=dev, generator=g)
    tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
    after = values()
    kept = (rows >= 0).nonzero().squeeze(1)
    key_of, grad_of = table_row[rows[kept].long()], grad[kept // 3].double()
    hot = key_of == 7                                    # (summed apart: index_add_ is slow where one row repeats)
    total = torch.zeros(known, dim, dtype=torch.float64, device=dev)
    total.index_add_(0, key_of[~hot], grad_of[~hot])
    total[7] = grad_of[hot].sum(dim=0)
    ref = before.double() - 0.05 * total / (total.pow(2).mean(dim=1, keepdim=True).sqrt() + 1e-6)
    assert ((after.double() - ref).abs() <= 2e-5 * (ref.abs() + 0.05)).all()
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()
