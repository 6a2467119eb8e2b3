"""The inference kernel with the streamed operand on bfloat16 rows that are not whole 16-byte groups: they move in words or, some
instances, in 16-byte vectors on word boundaries, where the vector a row ends in is another one in the last row and the last cluster.

Against the oracle: exact ranking (ties to 1e-5 exempt), one rounding of the result to bfloat16 (half a unit of 2^-8)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_26277_amd import binding, cat_apply

from parity_util import check_assignments_lazy, check_values, dev_matrix, f32_round, host_matrix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _streamed_operand():
    binding.debug_apply_kernel(3)  # this kernel or an error
    yield
    binding.debug_apply_kernel(0)


# words of a row past the last whole vector: 1, 2, 3 and none; rows that end in the first, a middle and the last vector of the lanes
@pytest.mark.parametrize("N,D,K", [(129, 522, 100), (128, 524, 110), (70, 526, 70), (130, 770, 40), (97, 1022, 64), (200, 1026, 33), (145, 1534, 128),
                                   (33, 1538, 17), (100, 2042, 50), (31, 2044, 30), (112, 2046, 100), (230, 1010, 200), (255, 1502, 250),
                                   (131, 294, 77), (100, 1126, 8), (65, 1126, 40)])
@pytest.mark.parametrize("alpha", [1.0, 0.6])
def test_against_the_oracle(N, D, K, alpha):
    rng = np.random.default_rng(N + D + K)
    cent = rng.standard_normal((K, D)) * 2
    label = rng.integers(0, K, N)
    label[-1], label[0] = K - 1, K - 1  # the last row and others in the last cluster
    x = torch.from_numpy(cent[label] + rng.standard_normal((N, D))).bfloat16().float().numpy()
    x[N // 2] = torch.from_numpy(0.5 * (cent[0] + cent[K - 1])).bfloat16().float().numpy()  # between two of them: measured in double
    cent, g, b = f32_round(cent), f32_round(rng.uniform(0.5, 1.5, (K, D))), f32_round(rng.standard_normal((K, D)))
    f = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda()
    out, a = cat_apply(dev_matrix(x, "bf16"), f(cent), f(g), f(b), alpha=alpha)
    a = a.cpu().numpy()
    want, o_a = oracle.apply(x, cent, g, b, alpha)
    check_assignments_lazy(a, o_a, x, cent, "labels")
    same = a == o_a
    assert N - same.sum() <= 1
    check_values(host_matrix(out)[same], want[same], 4e-3, "corrected")
