"""The reduction of rows wider than 256 elements keeps a few pairs in flight per wave, four of fp32 rows and two of bf16
ones: runs that end, begin and go on at every position of those, batches around multiples of them and of the smallest
tile, against an fp64 reduction."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dim", [512, 768, 1024])
def test_runs_at_every_position_of_the_rows_in_flight(dim, bf16):
    from paper_2209_07663_amd.binding import Table
    dev, known = torch.device("cuda:0"), 500
    for n in (1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 257, 1000, 9001):
        g = torch.Generator(device=dev).manual_seed(n + dim)
        tab = Table(1 << 12, dim, 5, bf16=bf16, max_ids=1 << 14, device=dev)
        all_keys = torch.arange(known, device=dev)
        all_rows = tab.mono_lookup_or_insert(all_keys, 0)
        keys = torch.cumsum((torch.rand(n, device=dev, generator=g) < 0.4).long(), 0) % known   # runs of 1 to about 10
        keys[n // 3: n // 2] = 3                                                                 # and a hot row
        rows = tab.mono_lookup_or_insert(keys, 1)
        offs = torch.arange(n + 1, device=dev)
        grad = torch.randn(n, dim, device=dev, generator=g)
        each = torch.arange(known + 1, device=dev)
        before = tab.mono_gather_pool(all_rows, each).double()
        tab.mono_apply_grad_adagrad(rows, offs, grad, 0.05, 1e-6)
        after = tab.mono_gather_pool(all_rows, each).double()
        total = torch.zeros(known, dim, dtype=torch.float64, device=dev).index_add_(0, keys, grad.double())
        ref = before - 0.05 * total / (total.pow(2).mean(dim=1, keepdim=True).sqrt() + 1e-6)
        # fp32: sums of up to 1500 terms and a 1-ulp root, relative to steps of about 0.05; bf16: half a unit of the
        # last of eight bits on top
        tol = 2e-5 * (ref.abs() + 0.05) + (2.0 ** -8 * ref.abs() if bf16 else 0.0)
        assert ((after - ref).abs() <= tol).all(), (n, float(((after - ref).abs() - tol).max()))
        tab.close()
