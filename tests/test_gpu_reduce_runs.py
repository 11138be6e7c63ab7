"""Gradient reduction where runs of one row's occurrences meet the borders of chunks, waves and tiles: runs of one
occurrence beside runs that fill a chunk, a wave, a tile and several of them, for every number of lanes that share a row;
against plain fp64 sums and Adagrad."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LR, EPS = 0.05, 1e-8
LENGTHS = [1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 4099]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dim", [4, 8, 16, 20, 32, 64, 128, 256, 512, 1024])
def test_runs_of_all_lengths(dim, bf16):
    from paper_2209_07663_amd.binding import Table
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(dim + bf16)
    for case in range(3):
        # (shuffled: the borders fall elsewhere in every run; case 1: one row only, and nothing but its run; case 2: a batch
        # large enough for the largest tiles)
        lengths = {0: LENGTHS, 1: [9000], 2: LENGTHS * 4 + [60000]}[case]
        lens = torch.tensor(lengths, device=dev)[torch.randperm(len(lengths), device=dev, generator=g)]
        keys = torch.repeat_interleave(torch.arange(len(lengths), dtype=torch.int64, device=dev), lens)
        if case == 2:
            keys = torch.cat([keys, torch.arange(1000, 1000 + (1 << 18) // max(1, dim // 32), dtype=torch.int64, device=dev)])
        n = keys.shape[0]
        keys = keys[torch.randperm(n, device=dev, generator=g)].contiguous()
        tab = Table(1 << 19, dim, 3, bf16=bf16, max_ids=n, max_bags=n, device=dev)
        rows = tab.mono_lookup_or_insert(keys, 0)
        one_each = torch.arange(n + 1, dtype=torch.int64, device=dev)
        bags = torch.cat([one_each[0:n:3], one_each[n:]])                  # bags of three, a shorter one at the end
        before = tab.mono_gather_pool(rows, one_each).double()             # the row of every occurrence
        grad = torch.rand((bags.shape[0] - 1, dim), device=dev, generator=g) + 0.25   # (no sum cancels)
        tab.mono_apply_grad_adagrad(rows, bags, grad, LR, EPS)
        got = tab.mono_gather_pool(rows, one_each).double()
        stored, at = torch.unique(keys, return_inverse=True)
        total = torch.zeros((stored.shape[0], dim), dtype=torch.float64, device=dev)
        total.index_add_(0, at, grad.double()[torch.arange(n, device=dev) // 3])
        count = torch.bincount(at).double()[:, None]
        move = LR * total / ((total ** 2).mean(1, keepdim=True).sqrt() + EPS)
        want = before - move[at]
        # sums of positive numbers: at most 256 additions in a row of a chunk, 16 of the scans, one per 8 tiles of the
        # run's pieces; the ratio of a sum and the root of its mean square doubles that, and the result is rounded once
        rel = 2 * (272 + count[at] / 256) * 2.0 ** -24
        assert ((got - want).abs() <= rel * move[at] + want.abs() * (2.0 ** -8 if bf16 else 2.0 ** -23)).all(), (case, dim)
        # a row's move says little of the length of its sum, its accumulator does: twice the error of the sums, and at
        # most twenty roundings of a mean of squares (four pieces of four elements a lane, six levels of lanes)
        dump = tab.mono_table_export()
        acc = (total ** 2).mean(1).cpu().numpy()
        assert (dump["keys"] == stored.cpu().numpy()).all()
        assert (abs(dump["acc"] - acc) <= (2 * (272 + count[:, 0].cpu().numpy() / 256) + 20) * 2.0 ** -24 * acc).all(), (case, dim)
        assert tab.mono_table_stats()["n_lost"] == 0
        tab.close()
