"""Every tile shape of the kernels with one workgroup per CU, with one to six 64-wide steps (fewer than the rings hold, as
many, and more) and ragged rows: the K and V rows, the attention output and the FFN output that the first step of a layer
leaves in its caches, against plain float64 sums.  Each case names the tiles that it is there for: Q | K, V-verify, output
projection, gate/up and down projection ("-": another kernel).

What a row goes through before each check is taken from the device, so that only one projection's roundings separate the two sides
(the attention output: Q's, the softmax and the output projection; the FFN output: norm, gate/up and down projection)."""
import ctypes

import pytest
import torch

from paper_2506_06295_amd import binding

pytestmark = pytest.mark.gpu

EPS, THETA = 1e-5, 10000.0


def _tile(launch, M, N, N0, K):
    cols = ctypes.c_int32()
    rows = binding.lib().dllmc_plan_tile(launch, M, N, N0, K, ctypes.byref(cols))
    return f"{rows}x{cols.value}" if rows else "-"


def _norm(x, g):
    return (x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + EPS) * g.double()).bfloat16().double()


def _rope(x, heads):
    """Pairs (t, t + 64) of every head of 128 turned by position * theta^(-t / 64)."""
    n = x.shape[0]
    t = torch.arange(64, dtype=torch.float64, device=x.device)
    ang = torch.arange(n, dtype=torch.float64, device=x.device)[:, None] * THETA ** (-t / 64)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    x = x.view(n, heads, 128)
    lo, hi = x[..., :64], x[..., 64:]
    return torch.cat((lo * c - hi * s, hi * c + lo * s), -1).view(n, heads * 128)


@pytest.mark.parametrize("M,d,H,G,m,tiles", [
    (265, 1024, 32, 32, 192, "128x128 192x64 128x128 128x64 128x128"),
    (1526, 1536, 32, 32, 1536, "192x256 128x256 256x128 128x96 192x128"),
    (265, 128, 32, 32, 128, "128x128 192x64 - 128x64 128x128"),
    (1548, 2560, 24, 8, 6144, "256x128 192x64 192x256 256x96 256x256"),
    (272, 64, 32, 32, 64, "128x128 192x64 - 128x64 -"),
    (314, 192, 32, 32, 128, "128x128 192x64 - 128x64 -"),
    (2061, 64, 32, 32, 2432, "192x256 192x256 - 192x128 -"),
    (545, 4096, 32, 32, 64, "192x128 - 128x256 128x64 128x128"),
    (2143, 192, 32, 32, 1536, "192x256 192x256 - 128x128 -"),
    (2248, 128, 32, 32, 3072, "192x256 192x256 128x128 256x128 -"),
    (585, 64, 32, 32, 6144, "192x128 192x64 - 128x128 -"),
    (671, 128, 24, 24, 3072, "192x128 192x64 - 128x96 -"),
    (642, 192, 24, 24, 3072, "192x128 192x64 - 128x96 -"),
    (792, 128, 32, 32, 2432, "256x128 - - 192x64 -"),
    (1166, 64, 20, 20, 3072, "256x128 - - 192x96 -"),
    (961, 192, 32, 16, 2432, "256x128 192x64 - 192x64 -"),
    (2894, 4096, 1, 1, 192, "- - 192x256 128x64 192x256"),
    (3195, 4096, 1, 1, 192, "- - 256x256 128x64 256x256"),
    (1547, 64, 32, 32, 6144, "256x256 - - 256x96 -"),
    (2679, 64, 12, 12, 2432, "128x256 - - 256x128 -"),
    (1539, 128, 32, 32, 3072, "256x256 - - 256x96 -"),
    (2662, 128, 12, 12, 1536, "128x256 - - 128x128 -"),
    (2562, 320, 12, 12, 1536, "128x256 - - 128x128 -"),
    (1632, 192, 32, 32, 3072, "256x256 - - 256x96 -"),
    (1740, 256, 32, 32, 2432, "256x256 - - 192x128 -"),
    (2320, 192, 24, 2, 3072, "128x256 - - 256x128 -"),
    (2062, 256, 32, 32, 6144, "192x256 192x256 128x128 192x96 128x128"),
    (378, 64, 6, 6, 6144, "- 192x64 - 128x96 -"),
    (985, 64, 2, 2, 2432, "- 192x64 - 192x64 -"),
    (293, 128, 1, 1, 12288, "- - 128x128 192x96 -"),
    (777, 256, 1, 1, 2432, "- - 128x128 192x64 -"),
    (1691, 128, 1, 1, 2432, "- - 128x128 192x128 -"),
    (198, 512, 1, 1, 12288, "- - 128x128 256x48 -"),
    (357, 192, 24, 24, 12288, "- 192x64 - 192x96 -"),
    (1071, 256, 1, 1, 6144, "- - 128x128 256x128 -"),
    (531, 192, 16, 16, 18944, "- 192x64 - 192x128 -"),
    (1155, 1536, 1, 1, 2432, "- - 128x128 256x64 128x128"),
    (1553, 2560, 6, 6, 192, "- 192x64 192x128 128x64 192x128"),
    (3106, 512, 32, 32, 192, "256x256 256x256 128x128 128x64 128x128"),
])
def test_first_step(M, d, H, G, m, tiles):
    dq, dkv = 128 * H, 128 * G
    assert " ".join([_tile(2, M, dq + dkv, dq, d), _tile(3, M, dkv, dkv, d), _tile(0, M, d, d, dq), _tile(1, M, m, m, d),
                     _tile(0, M, d, d, m)]) == tiles
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7 + d + m)
    make = lambda rows, cols, rms: (rms / cols ** 0.5 * torch.randn((rows, cols), generator=g, device="cuda")).bfloat16()
    w = {"wq": make(dq, d, 1.6), "wk": make(dkv, d, 1.6), "wv": make(dkv, d, 1.0), "wo": make(d, dq, 2.0),
         "w_gate": make(m, d, 1.6), "w_up": make(m, d, 1.0), "w_down": make(d, m, 2.0)}
    for k in ("attn_norm_g", "ffn_norm_g"):
        w[k] = (1 + 0.1 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    hid = torch.randn((1, M, d), generator=g, device="cuda").bfloat16()
    paging = None
    if M % 2:  # rows reach the caches through a row map
        per = -(-M // 16)
        order = torch.randperm(per + 3, generator=torch.Generator().manual_seed(M))[:per].reshape(1, per)
        paging = {"page_rows": 16, "pool_pages": per + 3, "page_table": order.tolist()}
    den = binding.CachedDenoiser(n_layers=1, d_model=d, n_q_heads=H, n_kv_heads=G, head_dim=128, d_ffn=m, batch=1,
                                 dtype="bf16", weights=[w], L_p=M - 32, L_r=32, rho=0.25, K_p=4, K_r=4, rms_eps=EPS,
                                 rope_theta=THETA, paging=paging)
    den.step(hid, 0)
    k, v, attn, ffn = (den.read_cache(0, i)[0].double() for i in range(4))
    den.close()
    x = hid[0].double()
    h = _norm(x, w["attn_norm_g"])
    # bf16 results: half a unit in the last place (2^-8 of the value); besides, an element of h may have been rounded to the other
    # side (float32 norm): two of the largest per row.  K: in either of a pair, and 2^-12 for the angles in float32.
    flip = lambda wt: 2.0 ** -7 * h.abs().amax(1, keepdim=True) * float(wt.abs().max())
    want = h @ w["wv"].double().t()
    assert bool(((v - want).abs() <= 1.001 * 2.0 ** -8 * want.abs() + flip(w["wv"])).all())
    want = _rope(h @ w["wk"].double().t(), G)
    turn = 2.0 ** -12 * want.abs().amax(1, keepdim=True)
    assert bool(((k - want).abs() <= 1.001 * 2.0 ** -8 * want.abs() + 1.5 * flip(w["wk"]) + turn).all())
    # attention from the cached K and V: scores of rms 2.5, whose last bits (2^-9 of q per element) move a probability by
    # less than 1 % each way; a row of Q that is wrong gives another row altogether
    q = _rope(h @ w["wq"].double().t(), H).bfloat16().double().view(M, H, 128)
    o = torch.empty((M, H, 128), dtype=torch.float64, device="cuda")
    for i in range(H):
        kv = slice(128 * (i * G // H), 128 * (i * G // H) + 128)
        p = torch.softmax(q[:, i] @ k[:, kv].t().contiguous() / 128 ** 0.5, -1)
        o[:, i] = p @ v[:, kv].contiguous()
    want = o.view(M, dq).bfloat16().double() @ w["wo"].double().t()
    assert float(((attn - want).norm(dim=1) / want.norm(dim=1)).max()) < 0.03
    # FFN from the device's residual stream: bf16 of h and of the product silu(gate) * up on either side (2^-8 of an
    # element now and then, averaged over m or d of them), the result rounded once
    h = _norm(x + attn, w["ffn_norm_g"])
    u = (torch.nn.functional.silu(h @ w["w_gate"].double().t()) * (h @ w["w_up"].double().t())).bfloat16().double()
    want = u @ w["w_down"].double().t()
    rms = float(want.pow(2).mean().sqrt())
    assert bool(((ffn - want).abs() <= 1.001 * 2.0 ** -8 * want.abs() + 0.02 * rms).all())


# (V-verify with its scores; 64-column tiles are those of 192 rows)
@pytest.mark.parametrize("rows,d,d_kv,tile", [
    (260, 64, 1024, "192x64"),
    (372, 128, 2048, "192x64"),
    (1030, 192, 1024, "192x64"),
    (519, 256, 2048, "192x64"),
    (519, 1024, 2048, "192x64"),
    (1030, 1024, 4096, "128x256"),
    (1051, 2048, 4096, "128x256"),
    (2052, 64, 4096, "192x256"),
    (2052, 128, 4096, "192x256"),
    (2052, 192, 4096, "192x256"),
    (4103, 256, 2048, "192x256"),
    (2052, 2048, 4096, "192x256"),
    (3074, 512, 4096, "256x256"),
    (3319, 448, 4096, "256x256"),
    (3074, 1024, 4096, "256x256"),
])
def test_scores(rows, d, d_kv, tile):
    assert _tile(3, rows, d_kv, d_kv, d) == tile and binding.lib().dllmc_plan_vverify(1, rows, d, d_kv) != 0
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + d)
    h = torch.randn((rows, d), generator=g, device="cuda").bfloat16()
    wv = (0.02 * torch.randn((d_kv, d), generator=g, device="cuda")).bfloat16()
    v = h.double() @ wv.double().t()
    cache = (v + 0.1 * torch.randn((rows, d_kv), generator=g, device="cuda").double()).bfloat16()
    old = cache.double()
    scores = binding.op_vverify("bf16", h, wv, cache)
    assert bool(((cache.double() - v).abs() <= 1.001 * 2.0 ** -8 * v.abs() + 2.0 ** -24 * d * float(v.abs().max())).all())
    new = cache.double()
    want = (new * old).sum(1) / (new.norm(dim=1) * old.norm(dim=1)).clamp(min=1e-8)
    assert float((scores.double() - want).abs().max()) < 2.0 ** -24 * d_kv ** 0.5 * 4  # as in the paths' test
