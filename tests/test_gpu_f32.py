"""Float32 models: the matrix-core kernels of the gathered linear map and of attention, and whole steps.

Tolerances of a linear map: a float32 sum of K products whose partial sums grow like sqrt(j) collects a
relative error of about 2^-24 sqrt(K / 6) in any order; the bar is 2^-24 sqrt(K) + 2^-23."""
import numpy as np
import pytest
import torch

from oracle import dllm_cache_oracle as O
from paper_2506_06295_amd import binding
from tests import parity_util as PU
from tests.parity_util import rel_err
from tests.test_gpu_step import MINI_DREAM, MINI_LLADA, run_schedule

pytestmark = pytest.mark.gpu


def check_linear(M, N, K, gather, offset=0):
    r = np.random.default_rng(M * 7 + N * 3 + K)
    total = M + 5
    a = r.standard_normal((total, K)).astype(np.float32)
    w = (0.05 * r.standard_normal((N, K))).astype(np.float32)
    buf = torch.zeros(total * K + offset, device="cuda")
    buf[offset:] = torch.from_numpy(a.ravel()).cuda()
    A = buf[offset:].view(total, K)
    idx = r.permutation(total)[:M].astype(np.int32) if gather else None
    got = binding.op_linear("f32", A if gather else A[:M], torch.from_numpy(w).cuda(),
                            None if idx is None else torch.from_numpy(idx).cuda()).cpu().numpy()
    want = (a[idx] if gather else a[:M]).astype(np.float64) @ w.astype(np.float64).T
    bar = 2.0 ** -24 * np.sqrt(K) + 2.0 ** -23
    assert rel_err(got, want) < bar
    assert np.max(np.abs(got - want)) < 8 * bar * np.sqrt(np.mean(want ** 2))


@pytest.mark.parametrize("M,N,K,gather", [
    (1, 1, 4, False),           # one lane's worth of everything
    (33, 31, 20, True),         # ragged tiles, contraction shorter than the four groups' first chunks
    (32, 32, 64, False),        # whole tiles
    (8, 512, 260, True),        # K % 16: the last chunk of the last group is half zero
    (40, 1024, 3072, True),     # few rows, long contraction: slices
    (64, 64, 32, False),        # one step
    (65, 130, 100, True),       # 64 x 64 tiles, ragged, K % 32
    (352, 2048, 1024, True),    # 64 x 64 tiles, slices
    (300, 1000, 356, True),     # ragged in every direction
    (700, 900, 44, False),
])
@pytest.mark.parametrize("force_s", [0, 1, 3])
def test_linear(M, N, K, gather, force_s):
    binding.set_gemm_tuning(force_s=force_s)
    try:
        check_linear(M, N, K, gather)
    finally:
        binding.set_gemm_tuning(force_s=0)


@pytest.mark.parametrize("M,N,K,offset", [(40, 70, 71, 0), (40, 70, 72, 1), (130, 65, 50, 2)])
def test_linear_rows_that_are_not_in_16_byte_pieces(M, N, K, offset):
    check_linear(M, N, K, True, offset)


def test_linear_non_finite_values_stay_in_their_rows_and_columns():
    a = torch.ones((70, 100), device="cuda")
    w = torch.ones((66, 100), device="cuda")
    a[3, 99], a[5, 0], w[65, 98] = float("inf"), float("nan"), float("-inf")
    out = binding.op_linear("f32", a, w).cpu().numpy()
    want = np.full((70, 66), 100.0)
    want[3], want[:, 65] = np.inf, -np.inf
    want[3, 65], want[5] = np.nan, np.nan
    assert np.array_equal(out, want.astype(np.float32), equal_nan=True)


@pytest.mark.parametrize("dtype,B,Mq,n,H_q,H_kv,d_h", [
    ("f32", 1, 1, 1, 1, 1, 64),        # one query, one key: three wavefronts have no keys
    ("f32", 1, 17, 16, 2, 1, 128),     # second query tile of one row, one whole block of keys
    ("f32", 2, 33, 65, 4, 2, 64),      # ragged, two blocks for some wavefronts and one for others
    ("f32", 1, 16, 300, 7, 1, 128),    # grouped KV heads, five blocks each, the last range shorter
    ("f32", 2, 100, 1000, 2, 2, 128),
    ("bf16", 2, 37, 130, 4, 2, 64),    # converted as it is multiplied
    ("bf16", 1, 16, 64, 1, 1, 64),
])
def test_attention(dtype, B, Mq, n, H_q, H_kv, d_h):
    """Scores of a few units: their float32 error 2^-24 sqrt(d_h) passes through exp unchanged, the sums over
    n add 2^-24 sqrt(n); bf16 results are rounded once (2^-9 at most per element, 2^-9 / sqrt(3) in the norm)."""
    r = np.random.default_rng(Mq * 7 + n)
    q, k, v = (r.standard_normal((B, rows, h * d_h)).astype(np.float32) * s
               for rows, h, s in ((Mq, H_q, 1.5), (n, H_kv, 1.0), (n, H_kv, 1.0)))
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    dq, dk, dv = (torch.from_numpy(x).cuda().to(t) for x in (q, k, v))
    got = binding.op_attention(dtype, dq, dk, dv, H_q, H_kv, d_h).float().cpu().numpy()
    bar = 2.0 ** -24 * (8 * np.sqrt(d_h) + np.sqrt(n)) + (2.0 ** -9 if dtype == "bf16" else 0.0)
    for b in range(B):
        want = O.attention(*(x[b].double().cpu().numpy() for x in (dq, dk, dv)), H_q, H_kv, d_h)
        assert rel_err(got[b], want) < bar


@pytest.mark.parametrize("dtype,n,d_h", [("f32", 1, 64), ("f32", 37, 128), ("f32", 48, 64), ("bf16", 65, 64)])
def test_attention_non_finite_values_stay_in_their_columns(dtype, n, d_h):
    """Values of the last key among others; no key past it may count, not even times zero."""
    r = np.random.default_rng(n)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v = (torch.from_numpy(0.3 * r.standard_normal((1, rows, 2 * d_h)).astype(np.float32)).to(t) for rows in (19, n, n))
    v[0, n - 1, 3], v[0, n - 1, d_h + 5], v[0, 0, 7], v[0, n // 2, 9] = float("inf"), float("-inf"), float("nan"), float("inf")
    got = binding.op_attention(dtype, q.cuda(), k.cuda(), v.cuda(), 2, 2, d_h).float().cpu().numpy()[0]
    want = O.attention(*(x[0].double().numpy() for x in (q, k, v)), 2, 2, d_h)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    fin = np.isfinite(want)
    assert np.array_equal(got[~fin], want[~fin].astype(np.float32), equal_nan=True)
    assert np.allclose(got[fin], want[fin], rtol=2.0 ** -7 if dtype == "bf16" else 1e-5, atol=1e-5 if dtype == "f32" else 1e-3)


@pytest.mark.parametrize("cfg", [MINI_LLADA.replace(dtype="f32"), MINI_DREAM.replace(dtype="f32", m=2436),
                                 MINI_LLADA.replace(dtype="f32", B=1, L_p=20, L_r=17, m=3000)],
                         ids=["mini_llada", "mini_dream", "few_rows"])
def test_schedule(cfg):
    """Fused gate/up in both kernels (few rows: four groups over the contraction; hundreds: 64 x 64 tiles) and
    in slices, FFN widths that leave ragged tiles; attention with and without grouped KV heads."""
    gpu, ora, st = run_schedule(cfg.replace(steps=4), stress=True)
    assert st.failed == 0, st.failures
    assert st.worst_rel <= 1e-4
    PU.compare_caches(cfg, gpu, ora, st)
    gpu.close()
