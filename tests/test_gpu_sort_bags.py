"""The bag of every occurrence, which the first pass of the sort finds: one bag, few long bags, one occurrence per bag,
and bags of one occurrence among many empty ones, in batches whose last unit is cut; exact sums of integers."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bags", ["one", "three", "each", "sparse"])
@pytest.mark.parametrize("n", [8193, 70001, (1 << 20) - 1, (1 << 20) + 5000])
def test_each_occurrence_takes_its_bags_gradient(n, bags):
    from paper_2209_07663_amd.binding import Table
    dev, dim = torch.device("cuda:0"), 4
    tab = Table(1 << 18, dim, 5, max_ids=1 << 22, max_bags=1 << 22, device=dev)
    keys = torch.arange(n, device=dev) % 100003
    rows = tab.mono_lookup_or_insert(keys, 0)
    if bags == "one":
        offs = torch.tensor([0, n], device=dev)
    elif bags == "three":
        offs = torch.tensor([0, 1, n - 1, n], device=dev)
    elif bags == "each":
        offs = torch.arange(n + 1, device=dev)
    else:                                             # two empty bags behind each
        offs = torch.minimum((torch.arange(3 * n + 1, device=dev) + 2) // 3, torch.tensor(n, device=dev))
    lengths = offs[1:] - offs[:-1]
    bag = torch.repeat_interleave(torch.arange(lengths.numel(), device=dev), lengths)
    grad = (torch.arange(lengths.numel(), device=dev) % 251 + 1).float()[:, None].expand(-1, dim).contiguous()
    before = tab.mono_gather_pool(rows, torch.arange(n + 1, device=dev))
    tab.mono_apply_grad_adagrad(rows, offs, grad, 0.5, 0.0)
    after = tab.mono_gather_pool(rows, torch.arange(n + 1, device=dev))
    total = torch.zeros(100003, dtype=torch.float64, device=dev).index_add_(0, keys, grad[bag, 0].double())
    acc = torch.zeros(1 << 18, dtype=torch.float64, device=dev)
    dump = tab.mono_table_export()
    acc[torch.from_numpy(dump["row"].astype("int64")).to(dev)] = torch.from_numpy(dump["acc"].astype("float64")).to(dev)
    assert torch.allclose(acc[rows.long()], total[keys] ** 2, rtol=1e-6, atol=0)   # every gradient arrived, once
    assert torch.allclose(after, before - 0.5, rtol=0, atol=1e-5)
    tab.close()


@pytest.mark.parametrize("n", [3000, 70000])
def test_more_bags_than_three_steps_of_the_search_tell_apart(n):
    """Just over 2^24 bags, most of them empty: a block of 256 threads looks for its first one in a fourth step.  (The
    blocks of 3000 occurrences then search the bags that they have not walked over for a while, those of 70000 walk over all.)"""
    from paper_2209_07663_amd.binding import Table
    dev, dim, bags = torch.device("cuda:0"), 4, (1 << 24) + 4099
    tab = Table(1 << 17, dim, 5, max_ids=1 << 25, max_bags=1 << 25, device=dev)
    g = torch.Generator(device=dev).manual_seed(n)
    bag = torch.cat([torch.randint(0, bags, (n - 2000,), device=dev, generator=g), torch.arange(800, device=dev),
                     bags - 1 - torch.arange(800, device=dev), torch.full((400,), bags // 2, device=dev)]).sort().values
    lengths = torch.bincount(bag, minlength=bags)
    offs = torch.zeros(bags + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lengths, 0, out=offs[1:])
    keys = torch.arange(n, device=dev)
    rows = tab.mono_lookup_or_insert(keys, 0)
    grad = (torch.arange(bags, device=dev) % 8191 + 1).float()[:, None].expand(-1, dim).contiguous()
    tab.mono_apply_grad_adagrad(rows, offs, grad, 0.5, 0.0)
    acc = torch.zeros(1 << 17, dtype=torch.float64, device=dev)
    dump = tab.mono_table_export()
    acc[torch.from_numpy(dump["row"].astype("int64")).to(dev)] = torch.from_numpy(dump["acc"].astype("float64")).to(dev)
    # (one key per occurrence: its accumulator is the square of its bag's number; whole numbers of 26 bits, rounded at each sum)
    assert torch.allclose(acc[rows.long()], grad[bag, 0].double() ** 2, rtol=2.0 ** -21, atol=0)
    assert tab.mono_table_stats()["n_lost"] == 0
    tab.close()
