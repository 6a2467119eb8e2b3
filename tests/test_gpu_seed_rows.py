"""The seeded rows that a fit starts from, against the host's walk of the same counter: clusters around a batch of draws and around
the number of workgroups that copy the rows, up to the largest number, with every row drawn (most draws repeat one) and with few.
Whole numbers: the centroids of a fit of no iterations are the rows themselves."""
import pytest
import torch

from paper_2509_26277_amd import binding, cat_fit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,D,K", [(1, 4, 1), (63, 2, 63), (300, 6, 64), (65, 10, 65), (5000, 300, 255), (256, 4, 256), (257, 34, 257),
                                   (4000, 18, 600), (1023, 4, 1023), (1024, 260, 1024), (60000, 8, 1024)])
def test_a_fit_of_no_iterations_returns_the_rows_drawn(N, D, K, dtype):
    x = torch.arange(N, device="cuda")[:, None] * 7 + torch.arange(D, device="cuda")[None] * 3
    x = (x % 251).to(dtype).contiguous()  # (whole numbers that either type holds)
    for seed in (0, 2 ** 63 + 11):
        r = cat_fit(x, x, K, 0, seed=seed)
        idx = torch.tensor(binding.cat_init_indices(N, K, seed), device="cuda")
        assert torch.equal(r["centroids"], x[idx].float())
