"""The head's reductions: inside the vocabulary projection (bf16, whole 128-column tiles, up to 640 rows), over
runs of 4096 logits, and in one run; final norm with and without 16-byte pieces."""
import numpy as np
import pytest
import torch

from paper_2506_06295_amd import binding, inputs as I
from tests.test_gpu_generate import head_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M,vocab,d,gather", [
    ("bf16", 1, 128, 64, False),       # one tile, one 64-wide step, one row
    ("bf16", 127, 384, 192, True),     # last row of a tile missing, K % 128
    ("bf16", 129, 1152, 4608, False),  # a second row tile of one row; norm rows wider than the registers hold
    ("bf16", 640, 256, 128, True),     # the most rows reduced inside the projection
    ("bf16", 641, 256, 128, True),     # logits and one run
    ("bf16", 641, 8320, 128, False),   # 256 x 256 / 128 x 128 tiles, three runs
    ("bf16", 6, 8193, 200, True),      # a vocabulary in no whole tiles: plain kernel, three runs, scalar loads
    ("bf16", 3, 300, 12, False),       # rows in no whole 16-byte pieces
    ("f32", 3, 9000, 8, False),        # room for two partial results per row: two long runs
    ("f32", 2, 9000, 4, True),         # room for one: a single run of 9000
    ("f32", 33, 4097, 64, False),      # a second run of a few logits
])
def test_head(dtype, M, vocab, d, gather):
    x0, conf, want_x0, want_conf, logits = head_case(dtype, M, vocab, d, gather)
    # logits differ by their last bf16 rounding of a normed element here and there (2^-8 of one of d terms of
    # rms 0.05): the token is the oracle's or within that of it
    band = 1e-4 if dtype == "f32" else 2e-3
    for i in range(M):
        assert logits[i, want_x0[i]] - logits[i, x0[i]] <= band
    assert np.allclose(conf, want_conf, rtol=5e-5 if dtype == "f32" else 5e-3, atol=0)


@pytest.mark.parametrize("dtype,M,vocab,d", [("bf16", 200, 1024, 128), ("f32", 7, 20000, 128), ("bf16", 5, 20000, 72)])
def test_equal_logits_go_to_the_lower_token(dtype, M, vocab, d):
    x0, _, want_x0, _, _ = head_case(dtype, M, vocab, d, False, dup=True)
    assert np.all(x0 < vocab // 2) and np.mean(x0 == want_x0) > 0.95
    x0, conf, _, _, _ = head_case(dtype, M, vocab, d, False, flat=True)
    assert np.all(x0 == 0) and np.allclose(conf, 1.0 / vocab, rtol=2e-5)


@pytest.mark.parametrize("M,vocab,d", [(700, 6400, 1024), (1030, 12800, 512), (2000, 3200, 4096)])
def test_equal_logits_of_many_rows(M, vocab, d):
    """Rows beyond those that the projection reduces itself: a hundred tokens over and over."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + vocab)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()
    x0, _ = binding.op_head("bf16", normal(M, d), torch.ones(d, device="cuda").bfloat16(),
                            (0.05 * normal(100, d)).repeat(vocab // 100, 1).contiguous(), 1e-5)
    assert bool(((x0 >= 0) & (x0 < 100)).all())


@pytest.mark.parametrize("L_r,vocab", [(60, 4100), (150, 4100), (192, 12300)])
def test_equal_logits_of_a_wide_model(L_r, vocab):
    """The closed loop of a model whose weights no cache holds, a vocabulary in no whole tiles: a hundred
    tokens over and over, the first of the equal ones wins in every row."""
    cfg = I.CONFIGS["llada8b"].replace(T=1, L_p=32, L_r=L_r, steps=4, vocab=vocab)
    den = binding.CachedDenoiser(
        n_layers=1, d_model=cfg.d, n_q_heads=cfg.H_q, n_kv_heads=cfg.H_kv, head_dim=cfg.d_h, d_ffn=cfg.m, batch=1,
        dtype=cfg.dtype, weights=I.device_weights(cfg), L_p=cfg.L_p, L_r=L_r, rho=cfg.rho, K_p=cfg.K_p, K_r=cfg.K_r,
        rms_eps=cfg.rms_eps, rope_theta=cfg.rope_theta)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab + L_r)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()
    gen = binding.Generator(den, normal(vocab + 1, cfg.d), torch.ones(cfg.d, device="cuda").bfloat16(),
                            (0.02 * normal(100, cfg.d)).repeat(vocab // 100, 1).contiguous(), cfg.steps)
    tokens = torch.randint(0, vocab, (1, cfg.n), generator=g, device="cuda").to(torch.int32)
    tokens[:, cfg.L_p:] = vocab
    gen.step(tokens, 0)
    x0 = gen.read()[0]
    assert bool(((x0 >= 0) & (x0 < 100)).all())
    gen.close()
    den.close()


@pytest.mark.parametrize("dtype,vocab", [("bf16", 512), ("bf16", 12000), ("f32", 12000)])
def test_tokens_that_cannot_occur(dtype, vocab):
    """Logits of minus infinity, whole tiles and runs of them: probability 0; nothing else changes."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    r = np.random.default_rng(vocab)
    d, M = 128, 9
    hidden = torch.from_numpy(1.0 + r.random((M, d), dtype=np.float32)).cuda().to(t)
    w = torch.from_numpy(0.05 * r.standard_normal((vocab, d), dtype=np.float32)).cuda().to(t)
    gain = torch.ones(d, device="cuda", dtype=t)
    cut = torch.zeros(vocab, dtype=torch.bool, device="cuda")
    cut[:140] = True
    cut[vocab // 2:] = True
    cut[200:300:7] = True
    w[cut] = float("-inf")
    x0, conf = binding.op_head(dtype, hidden, gain, w, 1e-5)
    keep = torch.nonzero(~cut).flatten()
    y0, yconf = binding.op_head(dtype, hidden, gain, w[keep].contiguous(), 1e-5)
    assert torch.equal(x0.long(), keep[y0.long()])
    assert torch.allclose(conf, yconf, rtol=1e-5, atol=0)
    w[:] = float("-inf")  # no token at all: the first one, and no probability (0 / 0)
    x0, conf = binding.op_head(dtype, hidden, gain, w, 1e-5)
    assert bool((x0 >= 0).all()) and bool((x0 < vocab).all())
