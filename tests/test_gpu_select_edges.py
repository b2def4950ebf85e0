"""Bottom-k selection around whole wavefronts of positions and around the length from which the histogram kernel
takes over; the order is that of the keys (-inf first, the two zeros equal, +inf, then NaN), ties lowest index first.
Integers: everything is exact."""
import numpy as np
import pytest
import torch

from paper_2506_06295_amd import binding

pytestmark = pytest.mark.gpu


def expected(scores, k):
    key = np.where(np.isnan(scores), np.float32(0), scores) + np.float32(0)
    order = np.lexsort((np.arange(scores.shape[1])[None].repeat(len(scores), 0), key, np.isnan(scores)))
    return np.sort(order[:, :k], axis=1)


@pytest.mark.parametrize("L", [1, 3, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2000])
@pytest.mark.parametrize("values", ["spread", "close", "two", "special"])
def test_select(L, values):
    r = np.random.default_rng(L)
    B = 3
    s = {"spread": lambda: r.uniform(-1, 1, (B, L)),
         "close": lambda: 1 - 1e-6 * r.integers(0, 40, (B, L)),       # neighbouring keys, many equal
         "two": lambda: r.integers(0, 2, (B, L)),
         "special": lambda: r.choice([-np.inf, np.inf, 0.0, -0.0, np.nan, 1e-45, -1e-45, 3.4e38, -3.4e38], (B, L)),
         }[values]().astype(np.float32)
    for k in sorted({0, 1, L // 4, L // 2, L - 1, L}):
        got = binding.op_select(torch.from_numpy(s).cuda(), k).cpu().numpy()
        assert np.array_equal(got, expected(s, k)), (L, k)
