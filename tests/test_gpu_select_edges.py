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


@pytest.mark.parametrize("L", [40, 64, 200, 512, 900])
def test_indices_over_the_scores(L):
    """One sequence's indices may take the place of its scores."""
    r = np.random.default_rng(L)
    for k in (1, L // 3, L):
        s = r.uniform(-1, 1, (1, L)).astype(np.float32)
        room = torch.from_numpy(s).cuda()
        rc = binding.lib().dllmc_op_select(room.data_ptr(), 1, L, k, room.data_ptr(),
                                           torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        assert np.array_equal(room.view(torch.int32).cpu().numpy()[:, :k], expected(s, k)), (L, k)
