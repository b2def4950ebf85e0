"""Gate/up with gates of every size, element by element.

The rows of the hidden state are multiples of unit vectors, the output projection is zero and the down projection picks
columns, so that row j's gate and up values are column j of the weights (times 32, exactly) and the cached FFN output holds
bf16(silu(gate) * up) itself: half a unit in the last place of bf16, 2^-8 of the value, and a few float32 roundings."""
import pytest
import torch

from paper_2506_06295_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,m", [
    (100, 1536),   # the weight-streaming kernel
    (256, 1536), (256, 3072), (700, 1536), (1024, 3072),  # tile kernels
])
def test_gates_of_every_size(M, m):
    d = 1024
    g = torch.Generator(device="cuda")
    g.manual_seed(M + m)
    kind = torch.randint(0, 5, (m, d), generator=g, device="cuda")
    r = torch.rand((m, d), generator=g, device="cuda")
    gate = torch.where(kind == 0, -88.5 + 8.5 * r,                       # exp(-gate) near the end of float32
           torch.where(kind == 1, -20 + 20 * r,
           torch.where(kind == 2, 20 * r,
           torch.where(kind == 3, -(10 ** (2 + 28 * r)), 10 ** (1 + 28 * r))))).bfloat16()
    up = ((1 + torch.rand((m, d), generator=g, device="cuda")) * 2.0 ** torch.randint(0, 9, (m, d), generator=g, device="cuda")).bfloat16()
    w_gate = gate / 32
    w_gate[m // 2, 0] = 3e38  # 32 of these are infinite
    pick = torch.arange(d, device="cuda") * m // d
    w = {k: (0.02 * torch.randn(s, generator=g, device="cuda")).bfloat16()
         for k, s in (("wq", (128, d)), ("wk", (128, d)), ("wv", (128, d)))}
    w["wo"] = torch.zeros((d, 128), device="cuda").bfloat16()
    w["attn_norm_g"] = w["ffn_norm_g"] = torch.ones(d, device="cuda").bfloat16()
    w["w_gate"], w["w_up"] = w_gate, up / 32
    w["w_down"] = torch.zeros((d, m), device="cuda").bfloat16()
    w["w_down"][torch.arange(d, device="cuda"), pick] = 1
    hid = torch.zeros((1, M, d), device="cuda").bfloat16()
    hid[0, torch.arange(M), torch.arange(M)] = 64
    den = binding.CachedDenoiser(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=128, d_ffn=m, batch=1,
                                 dtype="bf16", weights=[w], L_p=M - 8, L_r=8, rho=0.5, K_p=4, K_r=4, rms_eps=1e-5)
    den.step(hid, 0)
    got = den.read_cache(0, 3)[0].double()
    den.close()
    inf_at = int((pick == m // 2).nonzero()[0])
    assert float(got[0, inf_at]) == float("inf")
    got, gate, up = got[1:], gate[pick, 1:M].t().double(), up[pick, 1:M].t().double()  # (row 0: 0 times infinity elsewhere)
    want = torch.nn.functional.silu(gate) * up
    seen = gate >= -88.5
    assert bool(((got - want).abs() <= 1.0001 * 2.0 ** -8 * want.abs())[seen].all())
    # (exp(-gate) is infinite in float32: minus zero)
    assert bool((got.abs() <= 1.01 * want.abs())[~seen].all())
