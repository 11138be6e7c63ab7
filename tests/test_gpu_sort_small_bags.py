"""The bag of every occurrence in batches that one block sorts, and in the smallest that are split: one bag, few long bags, one
occurrence per bag, and bags of one occurrence among many empty ones, where the block's rounds and waves are cut; exact sums of
integers."""
import statistics

import pytest
import torch

from tests import test_gpu_sort_bags as large

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bags", ["one", "three", "each", "sparse"])
@pytest.mark.parametrize("n", [2, 64, 65, 1024, 1025, 4095, 4096, 4097, 4999, 8191, 8192])
def test_each_occurrence_of_a_small_batch_takes_its_bags_gradient(n, bags):
    large.test_each_occurrence_takes_its_bags_gradient(n, bags)


def test_a_long_bag_costs_no_more_than_many_short_ones():
    """4096 occurrences in one bag used to be numbered by one thread: many times the update of 4096 bags."""
    from paper_2209_07663_amd.binding import Table
    dev, n, dim = torch.device("cuda:0"), 4096, 16
    tab = Table(1 << 16, dim, 5, max_ids=n, device=dev)
    rows = tab.mono_lookup_or_insert(torch.arange(n, device=dev), 0)
    took = {}
    for bags in (1, n):
        offs = torch.arange(bags + 1, device=dev) * (n // bags)
        grad = torch.ones((bags, dim), device=dev)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                tab.mono_apply_grad_adagrad(rows, offs, grad, 0.1, 1e-8)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[bags] = statistics.median(times[2:])
    assert took[1] < 3 * took[n], took
    tab.close()
