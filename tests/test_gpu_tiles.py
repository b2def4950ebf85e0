"""Refresh steps of the models' widths (gate/up, V-verify and Q|K finished in the tile kernels' epilogues) at row counts
around whole tiles and rounds, against a context whose maps of fewer than 2^20 rows all go through
the weight-streaming kernel.

Same inputs, other orders of summation: elements may round to neighbouring bf16 values (2^-7 of the value), and
those flips spread a little behind the attention; a step of a tile multiplied with the wrong operands moves its rows
by 0.2 rms and more.  The bars are those of the 120-launch test of the 768-row launches."""
import pytest
import torch

from paper_2506_06295_amd import binding, inputs as I

pytestmark = pytest.mark.gpu


BASES = {name: I.CONFIGS[name] for name in ("llada8b", "dream7b")}
BASES["2560_wide"] = BASES["llada8b"].replace(d=2560, H_q=20, H_kv=20, m=1536)


# (V-verify: 0 split contraction, 1 / 2 / 3 tiles of 128, 256 and 192 rows, 4 64 x 64 tiles.  Which tiles the other launches take
# follows from estimates; the cases of test_gpu_tile_shapes name theirs.)
@pytest.mark.parametrize("base,L_p,L_r,v_way", [
    ("llada8b", 20, 180, 4),     # 200 rows
    ("llada8b", 129, 255, 0),    # 384 rows: two whole 192-row tiles
    ("llada8b", 129, 256, 0),    # 385
    ("llada8b", 320, 256, 0),    # 576: three
    ("llada8b", 513, 256, 0),    # 769: a fifth tile of one row
    ("llada8b", 900, 130, 0),    # 1030: six rows past whole tiles of 256
    ("llada8b", 1900, 147, 1),   # 2047: a ragged sixteenth tile
    ("llada8b", 2800, 273, 2),   # 3073: a thirteenth 256-row tile of one row
    ("dream7b", 700, 67, 0),     # 767 rows, grouped KV heads, an FFN width that 96 does not divide
    ("2560_wide", 800, 200, 3),  # 1000: a sixth 192-row tile of 40 rows
])
def test_full_refresh(base, L_p, L_r, v_way):
    cfg = BASES[base].replace(T=1, K_p=1, K_r=1, L_p=L_p, L_r=L_r)
    assert binding.lib().dllmc_plan_vverify(1, L_p + L_r, cfg.d, cfg.d_kv) == v_way
    ws = I.device_weights(cfg)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L_p * 1000 + L_r)
    make = lambda: binding.CachedDenoiser(
        n_layers=cfg.T, d_model=cfg.d, n_q_heads=cfg.H_q, n_kv_heads=cfg.H_kv, head_dim=cfg.d_h,
        d_ffn=cfg.m, batch=cfg.B, dtype=cfg.dtype, weights=ws, L_p=L_p, L_r=L_r, rho=cfg.rho,
        K_p=cfg.K_p, K_r=cfg.K_r, rms_eps=cfg.rms_eps, rope_theta=cfg.rope_theta)
    tiles = make()
    binding.set_gemm_tuning(tile_min_m=1 << 20, fat_min_m=1 << 20)
    try:
        plain = make()
    finally:
        binding.set_gemm_tuning(tile_min_m=192, fat_min_m=512)
    for i in range(4):
        hid = torch.randn(cfg.B, cfg.n, cfg.d, device="cuda", generator=gen).to(torch.bfloat16)
        a_out, _ = tiles.step(hid, i)
        c_out, _ = plain.step(hid, i)
        torch.cuda.synchronize()
        pairs = [(tiles.read_cache(0, w), plain.read_cache(0, w), 0.03 if w < 2 else 0.12) for w in range(4)]
        pairs.append((a_out, c_out, 0.12))
        for which, (a, c, slack) in enumerate(pairs):
            a, c = a.float(), c.float()
            rms = float(c.pow(2).mean().sqrt())
            excess = float(((a - c).abs() - 0.03 * c.abs()).max()) / rms
            assert excess <= slack, (i, which, excess)
    tiles.close()
    plain.close()


@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 1024, 4096, 512), ("bf16", 512, 512, 256), ("f32", 200, 256, 192)])
@pytest.mark.parametrize("over", ["a", "w"])
def test_result_over_an_operand(dtype, M, N, K, over):
    """A single slice goes straight to the result unless that lies over an operand."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    src = {"a": torch.randn((M, K), generator=g, device="cuda").to(dt),
           "w": (0.05 * torch.randn((N, K), generator=g, device="cuda")).to(dt)}
    want = binding.op_linear_static(dtype, src["a"], src["w"], torch.empty((M, N), device="cuda"))
    out = torch.empty(max(M * N, src[over].numel()), device="cuda")  # holds the operand, then the result
    held = out.view(dt)[:src[over].numel()].view(src[over].shape)
    held.copy_(src[over])
    ops = {**src, over: held}
    got = binding.op_linear_static(dtype, ops["a"], ops["w"], out[:M * N].view(M, N))
    assert torch.equal(got, want)


@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 1024, 4096, 512), ("f32", 200, 512, 64)])
@pytest.mark.parametrize("entry", ["static", "scratch"])
def test_result_over_rows_that_are_gathered(dtype, M, N, K, entry):
    """The rows that a gathered map reads may lie behind the first M of its operand, and the result over them."""
    dt, code = (torch.bfloat16, 1) if dtype == "bf16" else (torch.float32, 0)
    L = binding.lib()
    assert L.dllmc_plan_gemm_slices(code, M, N, N, K, 8 * M * N) == 1  # a single slice, in many tiles
    g = torch.Generator(device="cuda")
    g.manual_seed(M * N)
    w = (0.05 * torch.randn((N, K), generator=g, device="cuda")).to(dt)
    more = -(-M * N * 4 // (K * w.element_size()))  # rows that the result covers
    room = torch.empty((M + more) * K * w.element_size() // 4, device="cuda")
    a = room.view(dt).view(M + more, K)
    a.copy_(torch.randn((M + more, K), generator=g, device="cuda"))
    idx = (M + torch.randperm(more, generator=g, device="cuda")[:M]).to(torch.int32)
    want = binding.op_linear_static(dtype, a[idx.long()], w, torch.empty((M, N), device="cuda"))
    assert torch.equal(binding.op_linear(dtype, a, w, idx), want)
    out = room[room.numel() - M * N:].view(M, N)
    assert out.data_ptr() >= a[M].data_ptr()
    if entry == "static":
        binding.op_linear_static(dtype, a, w, out, idx)
    else:
        scratch = torch.empty(8 * M * N, device="cuda")
        assert L.dllmc_op_linear(code, a.data_ptr(), idx.data_ptr(), M, w.data_ptr(), N, K, out.data_ptr(),
                                 scratch.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(out, want)


@pytest.mark.parametrize("M,N,K,whole", [(448, 2048, 1024, True), (288, 2048, 2048, True), (333, 3072, 1024, True),
                                         (700, 2432, 896, True), (1024, 896, 2432, True), (64, 4096, 12288, False)])
def test_one_slice_where_a_slice_sum_costs_more(M, N, K, whole):
    """A second launch that adds slices counts against them: small maps go whole to the result, the scratch buffer stays
    as it was; long walks of few rows are split."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    a = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    w = (0.05 * torch.randn((N, K), generator=g, device="cuda")).bfloat16()
    out, scratch = torch.empty((M, N), device="cuda"), torch.full((8 * M * N,), 77.0, device="cuda")
    assert binding.lib().dllmc_op_linear(1, a.data_ptr(), None, M, w.data_ptr(), N, K, out.data_ptr(), scratch.data_ptr(),
                                         torch.cuda.current_stream().cuda_stream) == 0
    want = a.double() @ w.double().t()
    assert float((out.double() - want).norm() / want.norm()) < 2.0 ** -24 * K ** 0.5
    assert bool((scratch == 77.0).all()) == whole


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 448])
@pytest.mark.parametrize("M", [256, 301])
def test_fewer_steps_than_the_ring_holds(M, K):
    """256 x 256 tiles whose whole contraction is one to seven 64-wide steps.  Exact products, at most K float32 additions:
    K 2^-24 of the sum of their magnitudes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    a = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    w = torch.randn((512, K), generator=g, device="cuda").bfloat16()
    binding.set_gemm_tuning(fat_min_m=200)
    try:
        got = binding.op_linear("bf16", a, w).double()
    finally:
        binding.set_gemm_tuning(fat_min_m=512)
    want, bound = a.double() @ w.double().t(), K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t())
    assert bool(((got - want).abs() <= bound).all())


@pytest.mark.parametrize("H,rows", [(1, 256), (1, 700), (2, 1100), (3, 640)])
def test_narrow_models(H, rows):
    """Two to six steps in gate/up, Q|K, V-verify: 128 x 128 tiles at most, 64 + 64 columns in gate/up, against the streaming
    kernel, bars as above."""
    cfg = BASES["llada8b"].replace(T=1, K_p=1, K_r=1, L_p=rows - 90, L_r=90, d=128 * H, H_q=H, H_kv=H, m=1536)
    ws = I.device_weights(cfg)
    make = lambda: binding.CachedDenoiser(
        n_layers=1, d_model=cfg.d, n_q_heads=H, n_kv_heads=H, head_dim=128, d_ffn=cfg.m, batch=1, dtype=cfg.dtype,
        weights=ws, L_p=cfg.L_p, L_r=cfg.L_r, rho=cfg.rho, K_p=1, K_r=1, rms_eps=cfg.rms_eps, rope_theta=cfg.rope_theta)
    tiles = make()
    binding.set_gemm_tuning(tile_min_m=1 << 20, fat_min_m=1 << 20)
    try:
        plain = make()
    finally:
        binding.set_gemm_tuning(tile_min_m=192, fat_min_m=512)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    hid = torch.randn(1, rows, cfg.d, device="cuda", generator=gen).to(torch.bfloat16)
    a_out, c_out = tiles.step(hid, 0)[0], plain.step(hid, 0)[0]
    for a, c in [(tiles.read_cache(0, w), plain.read_cache(0, w)) for w in range(4)] + [(a_out, c_out)]:
        a, c = a.float(), c.float()
        assert float(((a - c).abs() - 0.03 * c.abs()).max()) <= 0.12 * float(c.pow(2).mean().sqrt())
    tiles.close()
    plain.close()


@pytest.mark.parametrize("H,m,L_p,L_r", [
    (8, 3072, 300, 90),     # 390 rows: 128-row tiles throughout
    (16, 3072, 900, 124),   # 1024: whole tiles of 128 and 256
    (32, 6144, 1100, 180),  # 1280: a seventh 192-row tile of 128 rows
    (16, 2432, 1400, 137),  # 1537: rows past whole tiles of 128, 192 and 256
    (24, 1536, 2700, 200),  # 2900
])
@pytest.mark.parametrize("paged", [False, True])
def test_shapes_between_the_two_widths(H, m, L_p, L_r, paged):
    """Steps that take the shapes between 128 x 128 and 256 x 256 somewhere, bars as above; paged
    caches reach the epilogues' rows through the row map."""
    cfg = BASES["llada8b"].replace(T=1, K_p=1, K_r=1, L_p=L_p, L_r=L_r, d=128 * H, H_q=H, H_kv=H, m=m)
    ws = I.device_weights(cfg)
    n = L_p + L_r
    per = -(-n // 16)
    paging = None
    if paged:
        order = torch.randperm(per + 3, generator=torch.Generator().manual_seed(n))[:per].reshape(1, per)
        paging = {"page_rows": 16, "pool_pages": per + 3, "page_table": order.tolist()}
    make = lambda: binding.CachedDenoiser(
        n_layers=1, d_model=cfg.d, n_q_heads=H, n_kv_heads=H, head_dim=128, d_ffn=m, batch=1, dtype=cfg.dtype, weights=ws,
        L_p=L_p, L_r=L_r, rho=cfg.rho, K_p=1, K_r=1, rms_eps=cfg.rms_eps, rope_theta=cfg.rope_theta, paging=paging)
    tiles = make()
    binding.set_gemm_tuning(tile_min_m=1 << 20, fat_min_m=1 << 20)
    try:
        plain = make()
    finally:
        binding.set_gemm_tuning(tile_min_m=192, fat_min_m=512)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    hid = torch.randn(1, n, cfg.d, device="cuda", generator=gen).to(torch.bfloat16)
    a_out, c_out = tiles.step(hid, 0)[0], plain.step(hid, 0)[0]
    for a, c in [(tiles.read_cache(0, w), plain.read_cache(0, w)) for w in range(4)] + [(a_out, c_out)]:
        a, c = a.float(), c.float()
        assert float(((a - c).abs() - 0.03 * c.abs()).max()) <= 0.12 * float(c.pow(2).mean().sqrt())
    tiles.close()
    plain.close()


@pytest.mark.parametrize("rows,d,d_kv", [(2500, 512, 4096), (2048, 512, 4096), (4609, 256, 4096), (1921, 1024, 4096)])
def test_vverify_wide_shapes(rows, d, d_kv):
    """V-verify of thousands of rows, whole and ragged tiles: bars of the paths' test."""
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    h = torch.randn((rows, d), generator=g, device="cuda").bfloat16()
    wv = (0.02 * torch.randn((d_kv, d), generator=g, device="cuda")).bfloat16()
    v = h.double() @ wv.double().t()
    cache = (v + 0.1 * torch.randn((rows, d_kv), generator=g, device="cuda").double()).bfloat16()
    old = cache.double()
    scores = binding.op_vverify("bf16", h, wv, cache)
    vb = v.bfloat16()
    assert float((cache != vb).double().mean()) < 0.01
    new = cache.double()
    want = (new * old).sum(1) / (new.norm(dim=1) * old.norm(dim=1)).clamp(min=1e-8)
    assert float((scores.double() - want).abs().max()) < 2.0 ** -24 * d_kv ** 0.5 * 4
