"""Pooling where the bags of a wave and the IDs in flight change: rows that share 4 to 64 lanes, bags whose average length
lies on either side of the rules, numbers of bags that end inside a wave; against a plain fp64 sum."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _batch(bags, average, space, dev):
    """Bags of `average` IDs on average, some empty, one long; IDs outside the space count as absent."""
    g = torch.Generator(device=dev).manual_seed(bags + average)
    lens = torch.randint(0, 2 * average + 1, (bags,), device=dev, generator=g)
    lens[bags // 2] += 100
    offs = torch.zeros(bags + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=offs[1:])
    return lens, offs, torch.randint(-1, space + 1, (int(offs[-1]),), device=dev, generator=g)


def _check(got, picked, lens):
    bag = torch.repeat_interleave(torch.arange(lens.shape[0], device=lens.device), lens)
    want = torch.zeros((lens.shape[0], picked.shape[1]), dtype=torch.float64, device=lens.device).index_add_(0, bag, picked)
    size = torch.zeros_like(want).index_add_(0, bag, picked.abs())
    # every fp32 addition rounds by at most 2^-24 of a partial sum, which the sum of the sizes bounds
    assert ((got.double() - want).abs() <= 2.0 ** -24 * (lens[:, None] + 2) * size).all()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dim", [16, 32, 64, 128, 256, 512])
def test_two_tables(dim, bf16):
    from paper_2209_07663_amd.binding import mono_qr_gather_pool
    dev, m = torch.device("cuda:0"), 9
    g = torch.Generator(device=dev).manual_seed(dim)
    tabs = [torch.randn((1 << m, dim), device=dev, generator=g).to(torch.bfloat16 if bf16 else torch.float32) for _ in range(2)]
    for bags, average in ((4099, 2), (4099, 4), (4099, 11), (4099, 13), (70001, 1), (110000, 2)):
        lens, offs, ids = _batch(bags, average, 1 << 2 * m, dev)
        got = mono_qr_gather_pool(tabs[0], tabs[1], ids, offs)
        inside = ((ids >= 0) & (ids < 1 << 2 * m))[:, None]
        at = ids.clamp(0, (1 << 2 * m) - 1)
        _check(got, (tabs[0].double()[at % (1 << m)] + tabs[1].double()[at >> m]) * inside, lens)


@pytest.mark.parametrize("dim,bf16", [(64, False), (64, True), (128, False), (256, False), (256, True), (512, False), (512, True),
                                      (132, False), (768, False), (768, True), (1024, False), (1024, True)])
def test_one_table(dim, bf16):
    from paper_2209_07663_amd.binding import Table
    dev = torch.device("cuda:0")
    tab = Table(1 << 12, dim, 3, bf16=bf16, max_ids=1 << 18, max_bags=1 << 17, device=dev)
    tab.mono_lookup_or_insert(torch.arange(3000, dtype=torch.int64, device=dev), 0)
    d = tab.mono_table_export()
    rows = torch.zeros((1 << 12, dim), dtype=torch.float64, device=dev)
    rows[torch.from_numpy(d["row"].astype("int64")).to(dev)] = torch.from_numpy(d["rows"]).to(dev).double()
    for bags, average in ((1000, 4), (8195, 2), (16387, 3), (33001, 1), (66003, 1)):
        lens, offs, at = _batch(bags, average, 1 << 12, dev)
        at = torch.where((at >= 3000) & (at < 1 << 12), -1, at)        # (rows that were never handed out hold anything)
        got = tab.mono_gather_pool(at.int(), offs)
        inside = ((at >= 0) & (at < 1 << 12))[:, None]
        _check(got, rows[at.clamp(0, (1 << 12) - 1)] * inside, lens)
    tab.close()


@pytest.mark.parametrize("longest", [1, 2])
@pytest.mark.parametrize("dim,bf16", [(4, False), (36, False), (64, True), (256, False), (512, True), (512, False)])
def test_bags_of_one_or_two(dim, bf16, longest):
    """Waves whose bags all hold at most `longest` IDs, some of them none, beside one whose first bag holds one more."""
    from paper_2209_07663_amd.binding import Table, mono_qr_gather_pool
    dev, m = torch.device("cuda:0"), 6
    g = torch.Generator(device=dev).manual_seed(dim + longest)
    tab = Table(1 << 12, dim, 3, bf16=bf16, max_ids=1 << 18, max_bags=1 << 17, device=dev)
    tab.mono_lookup_or_insert(torch.arange(3000, dtype=torch.int64, device=dev), 0)
    d = tab.mono_table_export()
    rows = torch.zeros((1 << 12, dim), dtype=torch.float64, device=dev)
    rows[torch.from_numpy(d["row"].astype("int64")).to(dev)] = torch.from_numpy(d["rows"]).to(dev).double()
    tabs = [torch.randn((1 << m, dim), device=dev, generator=g).to(torch.bfloat16 if bf16 else torch.float32) for _ in range(2)]
    for bags in (1, 63, 65, 4099, 70001):
        lens = torch.randint(0, longest + 1, (bags,), device=dev, generator=g)
        lens[bags // 2] = longest + (bags > 4000)
        offs = torch.zeros(bags + 1, dtype=torch.int64, device=dev)
        torch.cumsum(lens, 0, out=offs[1:])
        at = torch.randint(-1, 3000, (int(offs[-1]),), device=dev, generator=g)
        inside = (at >= 0)[:, None]
        _check(tab.mono_gather_pool(at.int(), offs), rows[at.clamp(min=0)] * inside, lens)
        ids = torch.where(at % 5 == 0, 1 << 2 * m, at)
        inside = ((ids >= 0) & (ids < 1 << 2 * m))[:, None]
        ids_in = ids.clamp(0, (1 << 2 * m) - 1)
        _check(mono_qr_gather_pool(tabs[0], tabs[1], ids, offs),
               (tabs[0].double()[ids_in % (1 << m)] + tabs[1].double()[ids_in >> m]) * inside, lens)
    tab.close()


@pytest.mark.parametrize("dim,bags", [(32, 12288 * 32 - 31), (64, 12288 * 16 - 16), (256, 12288 * 4 + 3)])
def test_two_tables_full_chip(dim, bags):
    """On either side of the size from which the rows of four IDs are held in flight together."""
    from paper_2209_07663_amd.binding import mono_qr_gather_pool
    dev, m = torch.device("cuda:0"), 9
    g = torch.Generator(device=dev).manual_seed(dim)
    tabs = [torch.randn((1 << m, dim), device=dev, generator=g) for _ in range(2)]
    for average in (1, 2, 5):
        lens, offs, ids = _batch(bags, average, 1 << 2 * m, dev)
        inside = ((ids >= 0) & (ids < 1 << 2 * m))[:, None]
        at = ids.clamp(0, (1 << 2 * m) - 1)
        _check(mono_qr_gather_pool(tabs[0], tabs[1], ids, offs),
               (tabs[0].double()[at % (1 << m)] + tabs[1].double()[at >> m]) * inside, lens)
