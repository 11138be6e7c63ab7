"""Updates of 4 K to a million pairs, which are split and sorted by bucket: both sides of every size, few rows in use, hot
rows, dropped occurrences and empty bags, and buckets that do not fit into a block's LDS at once; against fp64 sums and Adagrad."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LR, EPS, DIM = 0.05, 1e-8, 4
MOST_IN_LDS = 4096
LOSES_NO_PAIR = 16 * 2.0 ** -24


def _table(used, capacity):
    from paper_2209_07663_amd.binding import Table
    dev = torch.device("cuda:0")
    tab = Table(capacity, DIM, 5, max_ids=max(1 << 21, used), device=dev)
    for lo in range(0, used, 1 << 21):
        tab.mono_lookup_or_insert(torch.arange(lo, min(lo + (1 << 21), used), device=dev), 0)
    assert tab.mono_table_stats()["size"] == used           # rows 0 .. used - 1 are the ones in use
    return tab, dev


def _step(tab, dev, used, rows, lengths, acc):
    """One update of the table; `acc` (fp64, per row) goes along.  Compares every row in use and its accumulator.

    Gradients are 7, 8 or 9 times 2^-10: the sum of up to 2^20 of them is exact in fp32, in whatever order.  The mean of
    their four squares takes at most five roundings of 2^-24, and one more for every step before; a pair that is lost or
    taken twice changes it by 2 * 7 / 9 * 2^-20 or more.  (A row's move says little of the length of its sum: from an
    accumulator of zero it is the same for a sum and for half of it.)"""
    g = torch.Generator(device=dev).manual_seed(rows.shape[0])
    rows = torch.as_tensor(rows, dtype=torch.int32, device=dev)
    offs = torch.zeros(lengths.shape[0] + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lengths, 0, out=offs[1:])
    assert int(offs[-1]) == rows.shape[0]
    grad = torch.randint(7, 10, (lengths.shape[0], DIM), device=dev, generator=g).float() * 2.0 ** -10
    each, every = torch.arange(used + 1, device=dev), torch.arange(used, dtype=torch.int32, device=dev)
    before = tab.mono_gather_pool(every, each).double()
    tab.mono_apply_grad_adagrad(rows, offs, grad, LR, EPS)
    after = tab.mono_gather_pool(every, each).double()
    kept = (rows >= 0) & (rows < used)
    per_pair = grad.double()[torch.repeat_interleave(torch.arange(lengths.shape[0], device=dev), lengths)][kept]
    at = rows[kept].long()
    count = torch.bincount(at, minlength=used).double()[:, None]
    order = torch.argsort(at, stable=True)                                         # (index_add_ is slow where one row repeats)
    sums = torch.cat([torch.zeros((1, DIM), dtype=torch.float64, device=dev), per_pair[order].cumsum(0)])
    ends = torch.cumsum(count[:, 0].long(), 0)
    total = sums[ends] - sums[ends - count[:, 0].long()]
    acc += (total ** 2).mean(1)
    move = LR * total / (acc.sqrt()[:, None] + EPS)
    dump = tab.mono_table_export()
    stored = torch.zeros(used, dtype=torch.float64, device=dev)
    stored[torch.from_numpy(dump["row"].astype(np.int64)).to(dev)] = torch.from_numpy(dump["acc"].astype(np.float64)).to(dev)
    assert ((stored - acc).abs() <= LOSES_NO_PAIR * acc).all()
    # half of the accumulator's error, a root and a reciprocal of one unit each, three roundings of products and the row's own
    assert ((after - (before - move)).abs() <= 16 * 2.0 ** -24 * move + before.abs() * 2.0 ** -23 + 2.0 ** -40).all()
    assert tab.mono_table_stats()["n_lost"] == 0


def _bags(n, dev, seed):
    """Lengths of bags that hold n occurrences: 0 to 6 each, one of a thousand."""
    g = torch.Generator(device=dev).manual_seed(seed)
    lens = torch.randint(0, 7, (n,), device=dev, generator=g)
    lens[3] = 1000
    lens = lens[: int((torch.cumsum(lens, 0) <= n).sum())]
    return torch.cat([lens, torch.tensor([n - int(lens.sum()), 0, 0], device=dev)])


@pytest.mark.parametrize("used", [1, 2, 3, 17, 300, 5000, 300000])
def test_rows_in_use(used):
    tab, dev = _table(used, 1 << 20)
    acc = torch.zeros(used, dtype=torch.float64, device=dev)
    g = torch.Generator(device=dev).manual_seed(used)
    for n in (4097, 20001, 70000, 600000):
        rows = torch.randint(-1, used, (n,), device=dev, generator=g)
        _step(tab, dev, used, rows, _bags(n, dev, n), acc)
    tab.close()


@pytest.mark.parametrize("n", [4096, 4097, 65536, 65537, 131072, 131073, 524288, 524289, 1 << 20, (1 << 20) + 1])
def test_both_sides_of_every_size(n):
    used = 1 << 19
    tab, dev = _table(used, 1 << 20)
    acc = torch.zeros(used, dtype=torch.float64, device=dev)
    g = torch.Generator(device=dev).manual_seed(n)
    u = torch.rand(n, device=dev, generator=g, dtype=torch.float64)
    zipf = ((1 - u * (1 - float(used) ** -0.2)) ** -5).long().clamp_(1, used) - 1    # exponent 1.2: a fifth of the batch is one row
    zipf[n // 2:: 89] = -1
    _step(tab, dev, used, zipf, _bags(n, dev, 1), acc)
    _step(tab, dev, used, torch.full((n,), used - 1, device=dev), torch.ones(n, dtype=torch.int64, device=dev), acc)
    _step(tab, dev, used, torch.full((n,), -1, device=dev), torch.tensor([n], device=dev), acc)
    tab.close()


def _bucket(row, bits, buckets_log2, group_log2):
    """The bucket of a row, as the split computes it."""
    rest = bits - min(bits, buckets_log2)
    low = min(max(rest - 3, 0), group_log2)
    high = bits - low
    key = (((row >> low) * ((0x9E3779B1 >> (32 - high)) | 1)) & ((1 << high) - 1)) << low | (row & ((1 << low) - 1))
    return key >> rest


def _sampled(n, samples):
    i = np.arange(samples, dtype=np.uint64)
    first, last = n * i // samples, n * (i + 1) // samples
    return first + (((i * 0x9E3779B1) & 0xFFFFFFFF) * (last - first) >> np.uint64(32))


@pytest.mark.parametrize("n,buckets_log2,group_log2,samples", [(60000, 7, 2, 512), (120000, 8, 2, 1024), (300000, 9, 2, 1024),
                                                               (700000, 10, 0, 2048)])
def test_buckets_too_large_for_a_block(n, buckets_log2, group_log2, samples):
    """Many rows of one bucket, none of them often, and one that is but that no sample sees: together with the others of
    its bucket, alone, and more than a block holds by itself."""
    bits, rng = 18, np.random.default_rng(n)
    used = 1 << bits
    tab, dev = _table(used, 1 << 20)
    acc = torch.zeros(used, dtype=torch.float64, device=dev)
    all_rows = np.arange(used)
    bucket = _bucket(all_rows, bits, buckets_log2, group_log2)
    assert np.bincount(bucket, minlength=1 << buckets_log2).min() == used >> buckets_log2      # the hash is a bijection
    rows = rng.integers(0, used, n)
    free = np.setdiff1d(np.arange(n), _sampled(n, samples))                    # occurrences that no sample looks at
    free = rng.permutation(free)
    crowd, heavy, heavier = all_rows[bucket == 5][:200], all_rows[bucket == 5][200], all_rows[bucket == 6][0]
    rows[free[:9000]] = np.resize(crowd, 9000)
    rows[free[9000:12000]] = heavy
    rows[free[12000:17000]] = heavier
    assert (rows == heavier).sum() > MOST_IN_LDS and (_bucket(rows, bits, buckets_log2, group_log2) == 5).sum() > 2 * MOST_IN_LDS
    _step(tab, dev, used, rows, _bags(n, dev, 2), acc)
    tab.close()


@pytest.mark.parametrize("bits,pairs", [(18, 4096), (18, 4097), (18, 8191), (18, 8192), (18, 8193), (24, 4097), (24, 7500)])
def test_buckets_at_the_limits_of_a_block(bits, pairs):
    """One bucket of 4096 pairs, which are sorted as they are, of up to 8192, of which a word each is sorted, and of more,
    which are taken in pieces, as all of more than 4096 are where a word does not hold the key within the bucket (of 2^24
    rows in 16 buckets)."""
    n = 60000 if bits < 24 else 8192
    buckets_log2, used = (7, 1 << 18) if bits < 24 else (4, (1 << 23) + 11)
    rng = np.random.default_rng(pairs)
    tab, dev = _table(used, 1 << 24 if bits == 24 else 1 << 20)
    acc = torch.zeros(used, dtype=torch.float64, device=dev)
    bucket = _bucket(np.arange(used), bits, buckets_log2, 2)
    ours, others = np.flatnonzero(bucket == 3), np.flatnonzero(bucket != 3)
    rows = rng.choice(others, n)
    seen = _sampled(n, 512).astype(np.int64)
    free = rng.permutation(np.setdiff1d(np.arange(n), seen))
    some = np.concatenate([ours[rng.integers(0, ours.shape[0], 1500)], ours[rng.integers(0, 400, 6000)], np.full(1000, ours[7])])
    rows[free[:pairs]] = np.resize(rng.permutation(some), pairs)     # (none that a sample looks at: no row has a bin of its own)
    assert (bucket[rows] == 3).sum() == pairs
    for lengths in (_bags(n, dev, 3), torch.ones(n, dtype=torch.int64, device=dev)):
        _step(tab, dev, used, rows, lengths, acc)
    tab.close()
