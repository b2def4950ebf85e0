"""The weight-streaming kernel (bf16 maps of few rows, and of column counts that the tile kernels do not divide)
at the edges of its tiles, rings and slices.

bf16 products are exact in float32; a float32 sum of K of them is off by about 2^-24 sqrt(K / 6) of its size in any
order: the bar is 2^-24 sqrt(K) + 2^-23."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2506_06295_amd import binding, inputs as I
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


@pytest.mark.parametrize("M,N,K", [(333, 3072, 1024), (448, 2048, 1024), (100, 1000, 960), (64, 512, 1024)])
def test_sums_of_one_slice(M, N, K):
    """A result that is returned in float32: 16 steps in a single chain of additions are 1.28e-7 from 64 bits, in four chains
    7.7e-8 (a chain of n grows as sqrt(n); four of four and their sum make eight)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    a = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn((N, K), generator=g, device="cuda")).bfloat16()
    want = a.double() @ w.double().t()
    got = binding.op_linear("bf16", a, w).double()
    assert float((got - want).norm() / want.norm()) < 1.0e-7


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


FFN = I.Config("ffn", T=1, d=256, H_q=2, H_kv=2, d_h=128, m=1000, B=1, L_p=20, L_r=30, steps=2, rho=0.5, K_p=4, K_r=4,
               dtype="bf16", vocab=64)


# gate/up of a refresh, every workgroup shape that is chosen: 64, 128 and 192 rows x 16 to 80 columns of each matrix, last
# row and column tiles ragged; d = 256 is fewer steps than the ring has stages, d = 1024 more, from another start per tile
@pytest.mark.parametrize("M,m,d,rows,cols", [
    (50, 1000, 256, 64, 16), (50, 4136, 256, 64, 32), (50, 8208, 256, 64, 48), (50, 12312, 256, 64, 64),
    (50, 16424, 256, 64, 80), (384, 1358, 256, 128, 16), (100, 6176, 256, 128, 32), (100, 8208, 256, 128, 48),
    (100, 12312, 256, 128, 64), (100, 16424, 256, 128, 80), (150, 4136, 256, 192, 32), (150, 8208, 256, 192, 48),
    (150, 12312, 256, 192, 64), (150, 16424, 256, 192, 80),
    (50, 8208, 1024, 64, 48), (100, 6176, 1024, 128, 32), (150, 4136, 1024, 192, 32),
])
def test_gate_up_shapes(M, m, d, rows, cols):
    c = ctypes.c_int32()
    assert binding.lib().dllmc_plan_gate_up(M, m, d, ctypes.byref(c)) == rows and c.value == cols
    cfg = FFN.replace(m=m, d=d, L_p=M - 30)
    ws = I.device_weights(cfg)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + m + d)
    hid = torch.randn((1, M, d), generator=g, device="cuda").bfloat16()
    den = binding.CachedDenoiser(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=2, head_dim=128, d_ffn=m, batch=1,
                                 dtype="bf16", weights=ws, L_p=M - 30, L_r=30, rho=0.5, K_p=4, K_r=4,
                                 rms_eps=cfg.rms_eps, rope_theta=cfg.rope_theta)
    den.step(hid, 0)
    attn, ffn = den.read_cache(0, 2)[0], den.read_cache(0, 3)[0]
    w = {k: v.double() for k, v in ws[0].items()}
    x = (hid[0].float() + attn.float()).double()
    z = (x / (x.square().mean(1, keepdim=True) + cfg.rms_eps).sqrt() * w["ffn_norm_g"]).bfloat16().double()
    u = (torch.nn.functional.silu(z @ w["w_gate"].t()) * (z @ w["w_up"].t())).bfloat16().double()
    want = u @ w["w_down"].t()
    # three roundings of 2^-9 / sqrt(3); 16 columns of u left out or taken twice are sqrt(16 / m) > 2^-5 of the norm
    err = (ffn.double() - want).norm(dim=1) / want.norm(dim=1)
    assert float(err.max()) < 2.0 ** -7
    den.close()


@pytest.mark.parametrize("L_r,rho", [(100, 0.37), (128, 0.5), (128, 1.0), (180, 0.99)])  # 37, 64, 128, 178 rows
def test_weights_beyond_the_memory_side_cache(L_r, rho):
    """A model of more than 256 MB of weights streams them past the caches, one of a single layer does not: other loads
    and another walk over the contraction index, the same products.  Eleven layers that add nothing (zero output and
    down projections) behind the first make the one out of the other.

    Both add the same exact products in float32, so about 1e-3 of the elements of a bf16 result round the other way:
    2^-8 sqrt(1e-3) = 1.2e-4 per tensor, a few of which lie on the way to the output."""
    d, m, H, L_p = 1024, 3072, 8, 40
    g = torch.Generator(device="cuda")
    g.manual_seed(L_r)
    shapes = {"wq": (d, d), "wk": (d, d), "wv": (d, d), "wo": (d, d), "w_gate": (m, d), "w_up": (m, d), "w_down": (d, m)}
    first = {k: (0.02 * torch.randn(s, generator=g, device="cuda")).bfloat16() for k, s in shapes.items()}
    for k in ("attn_norm_g", "ffn_norm_g"):
        first[k] = torch.ones(d, device="cuda").bfloat16()
    rest = dict(first, wo=torch.zeros_like(first["wo"]), w_down=torch.zeros_like(first["w_down"]))
    h0 = torch.randn((1, L_p + L_r, d), generator=g, device="cuda").bfloat16()
    h1 = h0.clone()
    h1[:, L_p::3] = torch.randn_like(h1[:, L_p::3])
    got = []
    for layers in ([first], [first] + [rest] * 11):
        den = binding.CachedDenoiser(n_layers=len(layers), d_model=d, n_q_heads=H, n_kv_heads=H, head_dim=128, d_ffn=m,
                                     batch=1, dtype="bf16", weights=layers, L_p=L_p, L_r=L_r, rho=rho, K_p=99, K_r=99)
        den.step(h0, 0)
        out, n_sel = den.step(h1, 1)
        got.append([out, den.sel_idx[0, :, :n_sel].clone()] + [den.read_cache(0, w) for w in range(4)])
        den.close()
    assert torch.equal(got[0][1], got[1][1])
    for a, b in zip(got[0], got[1]):
        a, b = a.double(), b.double()
        assert float((a - b).norm() / a.norm()) < 1e-3
