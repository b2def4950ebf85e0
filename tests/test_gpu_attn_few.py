"""Attention of fewer than 128 queries (bf16, head width 128): the kernel whose wavefronts split the keys, at the edges
of its query tiles, key blocks and ranges, and the launches on both sides of the choice between kernels.

A bf16 result is rounded once: 2^-9 of an element at most, 2^-9 / sqrt(3) in the norm; the probabilities'
bf16 pairs (2^-17) and float32 sums are far below that."""
import numpy as np
import pytest
import torch

from oracle import dllm_cache_oracle as O
from paper_2506_06295_amd import binding
from tests.parity_util import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Mq,n,H_q,H_kv", [
    (1, 1, 1, 1, 1),          # one query, one key: three wavefronts without a block
    (1, 16, 32, 2, 2),        # one block
    (1, 17, 33, 2, 1),        # second query tile of one row, second block of one key
    (3, 33, 129, 4, 4),       # five blocks: two for the first wavefront
    (1, 64, 256, 32, 32),     # eight blocks, few queries per workgroup
    (2, 60, 300, 14, 2),
    (1, 62, 1254, 28, 4),     # key ranges and a merge
    (1, 20, 4096, 14, 2),     # eight or sixteen ranges
    (1, 127, 800, 8, 8),
    (4, 100, 1500, 32, 8),    # 64 queries per workgroup
    (1, 64, 768, 32, 32),     # the ranges of three blocks
    (6, 64, 200, 64, 64),     # 64-query tiles, whole ranges
])
@pytest.mark.parametrize("split_keys", [True, False])
def test_attention(B, Mq, n, H_q, H_kv, split_keys):
    r = np.random.default_rng(Mq * 7 + n)
    q, k, v = (torch.from_numpy(r.standard_normal((B, rows, h * 128)).astype(np.float32) * s).cuda().bfloat16()
               for rows, h, s in ((Mq, H_q, 1.5), (n, H_kv, 1.0), (n, H_kv, 1.0)))
    q[:, ::3] *= 0.05  # flat rows among peaky ones
    q[:, 1::5] *= 8    # and rows whose maximum moves far
    got = binding.op_attention("bf16", q, k, v, H_q, H_kv, 128, split_keys=split_keys).float().cpu().numpy()
    for b in range(min(B, 2)):
        want = O.attention(*(x[b].double().cpu().numpy() for x in (q, k, v)), H_q, H_kv, 128)
        assert rel_err(got[b], want) < 2.0 ** -9
        assert np.max(np.abs(got[b] - want)) <= 2.0 ** -8 * np.max(np.abs(want))


@pytest.mark.parametrize("B,Mq,n,H,split_keys", [
    (1, 33, 129, 4, False),      # 16 queries per workgroup
    (4, 40, 100, 32, False),     # 32
    (8, 48, 426, 32, False),     # 64
    (1, 51, 4608, 32, True),     # key ranges: a few workgroups do not walk all of them
    (1, 64, 768, 32, True),      # ranges of three blocks
    (8, 64, 250, 64, False),     # whole ranges, 64-query tiles
])
def test_result_at_eight_bytes(B, Mq, n, H, split_keys):
    """A result that is not 16-byte aligned comes from the same launches: the same bits, nothing beside them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, k, v = (torch.randn((B, rows, H * 128), generator=g, device="cuda").bfloat16() for rows in (Mq, n, n))
    want = binding.op_attention("bf16", q, k, v, H, H, 128, split_keys=split_keys)
    room = torch.zeros(q.numel() + 8, dtype=torch.bfloat16, device="cuda")
    out = room[4:4 + q.numel()]
    L = binding.lib()
    scratch = torch.empty(L.dllmc_op_attention_scratch_bytes(), dtype=torch.uint8, device="cuda") if split_keys else None
    rc = L.dllmc_op_attention(1, q.data_ptr(), B, Mq, k.data_ptr(), v.data_ptr(), n, H, H, 128, out.data_ptr(),
                              scratch.data_ptr() if split_keys else None, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(out, want.flatten())
    assert not room[:4].any() and not room[4 + q.numel():].any()
