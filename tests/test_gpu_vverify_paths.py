"""Every way through V-verify, at ragged sizes and around the choice between them: the split contraction with its row
kernel, 64 x 64 tiles in one launch, and the epilogue of the larger tile kernels.

bf16 rows are rounded once from float32 sums: isolated last-bit differences (2^-8 of an element) from another order
of summation; one of them moves a cosine of d_kv elements by at most ~2^-8 / sqrt(d_kv) * |v_i| / rms."""
import numpy as np
import pytest
import torch

from paper_2506_06295_amd import binding

pytestmark = pytest.mark.gpu


SPLIT, T128, T256, T192, T64 = range(5)


@pytest.mark.parametrize("rows,d,d_kv,way", [
    (64, 2048, 4096, SPLIT),
    (128, 2048, 4096, SPLIT),
    (251, 2048, 4096, T64),     # one round of the CUs, a ragged row tile
    (256, 2048, 4096, T64),
    (257, 2048, 4096, SPLIT),
    (416, 2048, 4096, SPLIT),
    (513, 2048, 4096, T192),    # a third row tile of 129 rows
    (1000, 2560, 2560, T192),   # a sixth row tile of 40 rows
    (899, 2048, 4096, T128),
    (900, 2048, 4096, T128),
    (1000, 2048, 512, T64),
    (50, 1024, 64, SPLIT),
    (3073, 512, 4096, T256),    # a thirteenth row tile of one row
    (1100, 1024, 64, T64),      # one column tile
])
def test_vverify(rows, d, d_kv, way):
    assert binding.lib().dllmc_plan_vverify(1, rows, d, d_kv) == way
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + d_kv)
    h = torch.randn((rows, d), generator=g, device="cuda").bfloat16()
    wv = (0.02 * torch.randn((d_kv, d), generator=g, device="cuda")).bfloat16()
    v = h.double() @ wv.double().t()
    old = (v + 0.3 * torch.rand((rows, 1), generator=g, device="cuda").double()
           * torch.randn((rows, d_kv), generator=g, device="cuda").double()).bfloat16()
    old[rows // 2] = 0
    cache = old.clone()
    scores = binding.op_vverify("bf16", h, wv, cache)
    vb = v.bfloat16()
    assert float((cache != vb).double().mean()) < 0.01
    assert float((cache.double() - vb.double()).norm() / vb.double().norm()) < 1e-3
    new = cache.double()
    want = (new * old.double()).sum(1) / (new.norm(dim=1) * old.double().norm(dim=1)).clamp(min=1e-8)
    assert float((scores.double() - want).abs().max()) < 2.0 ** -24 * np.sqrt(d_kv) * 4
    assert float(scores[rows // 2]) == 0.0


@pytest.mark.parametrize("rows,d", [(2048, 4096), (256, 2048)])
@pytest.mark.parametrize("over", ["h", "wv"])
def test_cache_over_an_operand(rows, d, over):
    """Cached rows that are also read as activations or weights, at sizes that take one launch otherwise.  Another
    order of summation: isolated last-bit differences, as above."""
    d_kv = d
    assert binding.lib().dllmc_plan_vverify(1, rows, d, d_kv) != SPLIT
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    h = torch.randn((rows, d), generator=g, device="cuda").bfloat16()
    wv = (0.02 * torch.randn((d_kv, d), generator=g, device="cuda")).bfloat16()
    old = (h if over == "h" else wv[:rows]).clone()
    want_cache = old.clone()
    want = binding.op_vverify("bf16", h, wv, want_cache)
    cache = h if over == "h" else wv[:rows]
    got = binding.op_vverify("bf16", h, wv, cache)
    assert float((cache != want_cache).double().mean()) < 0.01
    assert float((cache.double() - want_cache.double()).norm() / want_cache.double().norm()) < 1e-3
    assert float((got - want).abs().max()) < 2.0 ** -8 / np.sqrt(d_kv) * 4
