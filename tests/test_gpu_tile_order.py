"""The order in which the reduction takes its tiles where many gradients are shared by many occurrences: no result depends on
it.  The same pairs with so many empty bags behind them that there are fewer than two a bag are reduced in the plain order.
Gradients are small multiples of 2^-10, whose sums are exact in whatever order, so that both are the same to the bit; the
double-precision update is matched within fp32's rounding."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LR, EPS = 0.05, 1e-6


def _rows(kind, n, cap, g, dev):
    if kind == "one":
        return torch.full((n,), 7, dtype=torch.int32, device=dev)
    rows = torch.randint(0, cap // 2, (n,), dtype=torch.int32, device=dev, generator=g)
    if kind == "even":
        return rows
    hot = torch.randint(0, 60, (n,), dtype=torch.int32, device=dev, generator=g)
    rows = torch.where(torch.rand(n, device=dev, generator=g) < 0.7, hot, rows)
    if kind == "dropped":
        rows[torch.rand(n, device=dev, generator=g) < 0.3] = -1
    return rows


@pytest.mark.parametrize("bags,per,dim,bf16,kind", [
    (1 << 18, 4, 256, False, "hot"), (1 << 18, 4, 256, False, "even"), (1 << 18, 4, 256, False, "one"),
    (1 << 18, 5, 256, True, "dropped"), (1 << 16, 9, 1024, False, "hot"), ((1 << 21) + 3, 3, 64, True, "hot"),
    ((1 << 24) + 5, 3, 8, False, "dropped")])                   # (the last has more tiles than are held at a time)
def test_the_order_of_tiles_changes_nothing(bags, per, dim, bf16, kind):
    from paper_2209_07663_amd.binding import Table
    dev, cap, seed = torch.device("cuda:0"), 1 << 13, 3
    g = torch.Generator(device=dev).manual_seed(bags + dim)
    n = bags * per
    assert bags * dim * 4 >= 1 << 28 and n * dim * 4 >= 1 << 30 and n >= 2 * bags
    rows = _rows(kind, n, cap, g, dev)
    offsets = torch.arange(bags + 1, device=dev) * per
    behind = n // 2 - bags + 1                                  # empty bags that make it fewer than two IDs a bag
    grad = torch.randint(-4, 5, (bags + behind, dim), device=dev, generator=g, dtype=torch.int8).float().mul_(2.0 ** -10)
    keys = torch.arange(1, cap // 2 + 1, device=dev)
    dumps, tables = [], []
    for extra in (0, behind):
        tab = Table(cap, dim, seed, 1, 0, bf16, max_ids=n, max_bags=bags + behind, device=dev)
        place = tab.mono_lookup_or_insert(keys, 0)
        start = tab.mono_table_export()
        at = torch.empty(n, dtype=torch.int32, device=dev)
        used = rows >= 0
        at[used] = place[rows[used].long()]                      # the pairs by key: another table may number its rows otherwise
        at[~used] = -1
        off = torch.cat([offsets, torch.full((extra,), n, dtype=torch.int64, device=dev)])
        for _ in range(2):                                      # (and the counters are as they were)
            tab.mono_apply_grad_adagrad(at, off, grad[:bags + extra], LR, EPS)
        dumps.append(tab.mono_table_export())
        tab.close()
        del at
    ours, plain = dumps
    assert (ours["keys"] == plain["keys"]).all()
    count = np.bincount(rows[rows >= 0].cpu().numpy(), minlength=cap // 2)
    for k in ("rows", "acc"):
        assert (ours[k].view(np.uint32) == plain[k].view(np.uint32)).all(), k
    # against double precision: sum over the bags of each row (index_add of whole bags), the row-wise Adagrad twice
    total = torch.zeros((cap // 2, dim), dtype=torch.float64, device=dev)
    for lo in range(0, bags, 1 << 16):
        m = min(bags, lo + (1 << 16))
        r = rows[lo * per:m * per].view(m - lo, per)
        for j in range(per):
            ok = r[:, j] >= 0
            total.index_add_(0, r[ok, j].long(), grad[lo:m][ok].double())
    total = total.cpu().numpy()
    acc, w = np.zeros(cap // 2), start["rows"].astype(np.float64)
    most = np.abs(w)
    for _ in range(2):
        acc += (total ** 2).mean(1)
        w = w - LR * total / (np.sqrt(acc) + EPS)[:, None]
        most = np.maximum(most, np.abs(w))
    # the sum over a row's squares, its root and reciprocal: some ten roundings of 2^-24, of a step of at most
    # LR * sqrt(dim); a bf16 row (eight significant bits) is rounded twice, by at most
    # 2^-8 of itself each time
    tol = 2.0 ** -20 * (most + LR * dim ** 0.5) + (2 * 2.0 ** -8 * 1.01 * most if bf16 else 0.0)
    assert np.all(np.abs(ours["rows"] - w) <= tol)
    assert np.all(np.abs(ours["acc"] - acc) <= 2.0 ** -20 * acc)
    assert count.sum() == 0 or acc.max() > 0
