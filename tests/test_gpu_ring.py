"""The weight-streaming kernel (bf16 maps of few rows, and of column counts that the tile kernels do not divide)
at the edges of its tiles, rings and slices.

bf16 products are exact in float32; a float32 sum of K of them is off by about 2^-24 sqrt(K / 6) of its size in any
order: the bar is 2^-24 sqrt(K) + 2^-23."""
import numpy as np
import pytest
import torch

from paper_2506_06295_amd import binding
from tests import parity_util as PU
from tests.test_gpu_step import MINI_DREAM, MINI_LLADA, run_schedule

pytestmark = pytest.mark.gpu


def check(M, N, K, gather, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + M * 7 + N * 3 + K)
    a = torch.randn((M + 3, K), generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn((N, K), generator=g, device="cuda")).bfloat16()
    idx = torch.randperm(M + 3, generator=g, device="cuda")[:M].to(torch.int32) if gather else None
    got = binding.op_linear("bf16", a if gather else a[:M], w, idx)
    want = (a[idx.long()] if gather else a[:M]).double() @ w.double().t()
    bar = 2.0 ** -24 * np.sqrt(K) + 2.0 ** -23
    d = got.double() - want
    assert float(d.norm() / want.norm()) < bar
    assert float(d.abs().max()) < 8 * bar * float(want.square().mean().sqrt())


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 64),          # one step, one row, one column
    (64, 64, 192),       # fewer steps than stages
    (63, 72, 576),       # the ring wraps once; ragged rows and columns
    (65, 4096, 1024),    # a second row block
    (128, 200, 4160),    # 65 steps; columns no multiple of 16
    (129, 1000, 512),    # three row blocks
    (191, 136, 2432),
    (250, 1000, 832),    # rows of the tile kernels, columns that they do not divide
    (700, 40, 64),
    (62, 3584, 18944),   # eight slices of 37 steps
])
@pytest.mark.parametrize("gather", [False, True])
def test_linear(M, N, K, gather):
    check(M, N, K, gather)


@pytest.mark.parametrize("force_s", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("K", [64, 128, 448, 512, 576, 1088])
def test_slices_and_step_counts(K, force_s):
    """Slices of one step to more than twice the stages, the last one shorter."""
    binding.set_gemm_tuning(force_s=force_s)
    try:
        check(40, 128, K, True)
        check(100, 128, K, False)
    finally:
        binding.set_gemm_tuning(force_s=0)


@pytest.mark.parametrize("cfg", [
    MINI_LLADA.replace(B=1, m=2440),               # gate/up columns no multiple of 16 (down: the plain kernel)
    MINI_LLADA.replace(B=1, L_p=30, L_r=190, m=1600),  # 190 rows on a refresh: three row blocks, Q|K and gate/up
    MINI_DREAM.replace(L_r=260, rho=0.5, m=1216),  # 130 recomputed rows
], ids=["ffn_2440", "190_rows", "130_rows"])
def test_schedule(cfg):
    gpu, ora, st = run_schedule(cfg.replace(steps=4), stress=True)
    assert st.failed == 0, st.failures
    assert st.worst_rel <= 2e-2
    PU.compare_caches(cfg, gpu, ora, st)
    gpu.close()
