"""The work that a program has this framework do, as cases that can be timed and checked.

A case is one call (or one short run of calls) of the public entry points of
`paper_2506_06295_amd.binding` on inputs drawn from a seed:

* ``step``       denoising steps of a `CachedDenoiser`, the call the framework exists for.  ``mode``:
                 ``adaptive``  two adaptive steps (the update ratio's share of the response rows is
                               recomputed, everything else comes from the caches),
                 ``prompt``    the same with the prompt refreshed in both steps,
                 ``response``  a response refresh,
                 ``full``      step 0 of a generation (prompt and response; also the uncached forward).
                 Full depth repeats the same layer 28 to 32 times, so one to three layers stand for it.
* ``head``       `op_head`: final norm, vocabulary projection, greedy token and its confidence for the
                 rows that are still masked.
* ``attention``  `op_attention`: queries against a whole cached sequence.
* ``linear``     `op_linear`: a gathered linear map.
* ``vverify``    `op_vverify`, twice, with two states of the response in turn.
* ``select``     `op_select`: the bottom-k rows of a batch of scores.

Models: the LLaDA-8B and Dream-7B shapes of the benchmark, the small shapes of the tests, and the float32
toy.  Weights are N(0, 0.02), token embeddings N(0, 1), as everywhere in this repository.
"""
import math

import torch

from paper_2506_06295_amd import binding

# n_q_heads, n_kv_heads, head_dim, d_model, d_ffn, vocab
MODELS = {
    "toy": (4, 4, 64, 256, 704, 1024),
    "mini_llada": (8, 8, 128, 1024, 3072, 4096),
    "mini_dream": (7, 1, 128, 896, 2432, 4096),
    "llada8b": (32, 32, 128, 4096, 12288, 126464),
    "dream7b": (28, 4, 128, 3584, 18944, 152064),
}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
EPS, THETA = 1e-5, 10000.0
NEVER = 10 ** 9  # a refresh interval that no run reaches
WEIGHTS = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


def _step(model, mode, L_p, L_r, rho=0.25, B=1, layers=2, dtype="bf16", paged=False):
    return {"op": "step", "model": model, "mode": mode, "dtype": dtype, "layers": layers, "B": B,
            "L_p": L_p, "L_r": L_r, "rho": rho, "paged": paged}


def listed():
    cases = [
        # the smallest calls: a float32 model of two narrow layers, where launches and latency are all
        ("toy_f32_adaptive", _step("toy", "adaptive", 64, 32, dtype="f32")),
        # a float32 model of ordinary width: reference and debugging runs, first step of a generation
        ("mini_f32_full", _step("mini_llada", "full", 96, 80, B=2, dtype="f32")),
        # the headline workload, its three step kinds: 53, 9 and 1 of the 64 steps of a generation
        ("llada8b_adaptive", _step("llada8b", "adaptive", 512, 256)),
        ("llada8b_response", _step("llada8b", "response", 512, 256)),
        ("llada8b_full", _step("llada8b", "full", 512, 256)),
        # grouped KV heads, a ragged prompt and an odd response length: a served request
        ("dream7b_adaptive_ragged", _step("dream7b", "adaptive", 1003, 251)),
        # a long document: the first step over its whole prompt
        ("llada8b_long_full", _step("llada8b", "full", 4096, 512, rho=0.1, layers=1)),
        # sixteen sequences in one call
        ("llada8b_b16_adaptive", _step("llada8b", "adaptive", 512, 256, B=16, layers=1)),
        # the head half-way through a response, and at its end when few positions are left
        ("head_llada8b", {"op": "head", "model": "llada8b", "M": 100}),
        ("head_dream7b_last", {"op": "head", "model": "dream7b", "M": 4}),
        # an adaptive step's queries against a long cached prompt
        ("attention_long_prompt", {"op": "attention", "dtype": "bf16", "B": 1, "Mq": 51, "n": 4608,
                                   "H_q": 32, "H_kv": 32, "d_h": 128}),
        # a projection of gathered rows called by itself
        ("linear_gathered", {"op": "linear", "dtype": "bf16", "M": 333, "N": 4096, "K": 4096}),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = max(_cost(c) for c in listed())
    while True:
        case = _draw_any(rng)
        if _cost(case) <= largest:
            return case


def _draw_any(rng):
    op = rng.choice(["step"] * 6 + ["head", "head", "attention", "attention", "linear", "vverify", "select"])
    if op == "step":
        model = rng.choice(["toy", "mini_llada", "mini_dream", "llada8b", "llada8b", "dream7b", "dream7b"])
        wide = model in ("llada8b", "dream7b")
        dtype = "f32" if model == "toy" or (not wide and rng.random() < 0.5) else "bf16"
        L_p, L_r = (_log_int(rng, 64, 4096), _log_int(rng, 32, 512)) if wide else (_log_int(rng, 16, 200), _log_int(rng, 16, 130))
        return _step(model, rng.choice(["adaptive", "adaptive", "prompt", "response", "full"]), L_p, L_r,
                     rho=rng.choice([0.1, 0.25, 0.25, 0.5]), B=rng.choice([1, 1, 2, 4, 8] if wide else [1, 2]),
                     layers=1 if wide else rng.choice([1, 2, 3]), dtype=dtype, paged=rng.random() < 0.15)
    if op == "head":
        return {"op": "head", "model": rng.choice(["llada8b", "dream7b", "mini_llada"]), "M": _log_int(rng, 1, 256)}
    if op == "attention":
        H_q, H_kv, d_h = MODELS[rng.choice(["llada8b", "dream7b", "mini_dream"])][:3]
        return {"op": "attention", "dtype": "bf16", "B": rng.choice([1, 1, 2, 4]), "Mq": _log_int(rng, 8, 600),
                "n": _log_int(rng, 100, 4608), "H_q": H_q, "H_kv": H_kv, "d_h": d_h}
    if op == "linear":
        d, m = MODELS[rng.choice(["mini_llada", "mini_dream", "llada8b", "dream7b"])][3:5]
        N, K = rng.choice([(d, d), (m, d), (d, m)])
        dtype = "f32" if d <= 1024 and rng.random() < 0.5 else "bf16"
        return {"op": "linear", "dtype": dtype, "M": _log_int(rng, 1, 512 if dtype == "f32" else 2048), "N": N, "K": K}
    if op == "vverify":
        return {"op": "vverify", "model": rng.choice(["mini_llada", "llada8b", "dream7b"]), "rows": _log_int(rng, 16, 2048)}
    L = _log_int(rng, 32, 4096)
    return {"op": "select", "B": rng.choice([1, 2, 4, 8, 16]), "L": L, "k": max(1, int(L * rng.choice([0.1, 0.25, 0.5])))}


# ---------------------------------------------------------------------------------------- inputs

def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    for k in key:
        seed = (seed * 1000003 + k) % (2 ** 61 - 1)
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, std=1.0, mean=0.0):
    return (mean + std * torch.randn(shape, generator=g, device="cuda")).to(dtype)


def _layer(case, seed, l):
    H_q, H_kv, d_h, d, m, _ = MODELS[case["model"]]
    dt = DTYPES[case["dtype"]]
    shapes = {"wq": (H_q * d_h, d), "wk": (H_kv * d_h, d), "wv": (H_kv * d_h, d), "wo": (d, H_q * d_h),
              "w_gate": (m, d), "w_up": (m, d), "w_down": (d, m)}
    g = _gen(seed, 1, l)
    w = {k: _normal(g, shapes[k], dt, 0.02) for k in WEIGHTS}
    for k in ("attn_norm_g", "ffn_norm_g"):
        w[k] = _normal(g, (d,), dt, 0.1, 1.0)
    return w


def _k(case):
    return int(math.floor(case["rho"] * case["L_r"] + 1e-6))


def _hiddens(case, seed):
    """Two states of the embedded sequence that differ in exactly the rows an adaptive step recomputes: as many
    response tokens per sequence have changed.  Returns (first, second, changed [B, k] ascending positions)."""
    B, L_p, L_r, k = case["B"], case["L_p"], case["L_r"], _k(case)
    d, dt = MODELS[case["model"]][3], DTYPES[case["dtype"]]
    g = _gen(seed, 2)
    first = _normal(g, (B, L_p + L_r, d), dt)
    new = _normal(g, (B, k, d), dt)
    pos = torch.argsort(torch.rand((B, L_r), generator=g, device="cuda"), dim=1)[:, :k].sort(dim=1).values + L_p
    second = first.scatter(1, pos[:, :, None].expand(B, k, d), new)
    return first, second, pos


def _head_inputs(case, seed):
    d, vocab = MODELS[case["model"]][3], MODELS[case["model"]][5]
    M, dt = case["M"], torch.bfloat16
    g = _gen(seed, 3)
    lm = _normal(g, (vocab, d), dt, 0.02)
    gain = _normal(g, (d,), dt, 0.1, 1.0)
    rows_all = 2 * M + 1
    # rows lean towards one token each, as a trained model's do: confidences from a few per cent to nearly one
    tok = torch.randint(0, vocab, (rows_all,), generator=g, device="cuda")
    # (a lift of one would raise the token's logit by 0.02 * d)
    lift = (9.0 + 9.0 * torch.rand((rows_all, 1), generator=g, device="cuda")) / (0.02 * d)
    if vocab < 10000:
        lift = 0.7 * lift
    hid = torch.sqrt(1 - lift * lift) * torch.randn((rows_all, d), generator=g, device="cuda") + lift * lm[tok].float() / 0.02
    rows = torch.randperm(rows_all, generator=g, device="cuda")[:M].sort().values.to(torch.int32)
    return (3.0 * hid).to(dt), gain, lm, rows


def _attention_inputs(case, seed):
    B, Mq, n, d_h, dt = case["B"], case["Mq"], case["n"], case["d_h"], DTYPES[case["dtype"]]
    g = _gen(seed, 4)
    q = _normal(g, (B, Mq, case["H_q"] * d_h), dt, 1.3)
    k = _normal(g, (B, n, case["H_kv"] * d_h), dt, 1.3)
    v = _normal(g, (B, n, case["H_kv"] * d_h), dt, 1.3)
    return q, k, v


def _linear_inputs(case, seed):
    g = _gen(seed, 5)
    dt = DTYPES[case["dtype"]]
    a = _normal(g, (2 * case["M"] + 3, case["K"]), dt)
    w = _normal(g, (case["N"], case["K"]), dt, 0.02)
    rows = torch.randperm(a.shape[0], generator=g, device="cuda")[:case["M"]].sort().values.to(torch.int32)
    return a, w, rows


def _vverify_inputs(case, seed):
    H_q, H_kv, d_h, d, _, _ = MODELS[case["model"]]
    g = _gen(seed, 6)
    first = _normal(g, (case["rows"], d), torch.bfloat16)
    # the response drifts, a few rows by much
    drift = torch.rand((case["rows"], 1), generator=g, device="cuda") ** 4
    second = (first.float() + drift * torch.randn((case["rows"], d), generator=g, device="cuda")).to(torch.bfloat16)
    wv = _normal(g, (H_kv * d_h, d), torch.bfloat16, 0.02)
    return first, second, wv


def _scores(case, seed):
    # cosines of cached and new rows: most close to 1
    return 1.0 - torch.rand((case["B"], case["L"]), generator=_gen(seed, 7), device="cuda") ** 3


# ---------------------------------------------------------------------------------------- prepare, run

def prepare(case, seed):
    op = case["op"]
    if op == "step":
        H_q, H_kv, d_h, d, m, _ = MODELS[case["model"]]
        B, n = case["B"], case["L_p"] + case["L_r"]
        K_p = 1 if case["mode"] == "prompt" else NEVER
        K_r = 1 if case["mode"] == "response" else NEVER
        paging = None
        if case["paged"]:
            per = -(-n // 16)
            order = torch.randperm(B * per + 8, generator=_gen(seed, 8), device="cuda")[:B * per].reshape(B, per)
            paging = {"page_rows": 16, "pool_pages": B * per + 8, "page_table": order.tolist()}
        den = binding.CachedDenoiser(n_layers=case["layers"], d_model=d, n_q_heads=H_q, n_kv_heads=H_kv, head_dim=d_h,
                                     d_ffn=m, batch=B, dtype=case["dtype"],
                                     weights=[_layer(case, seed, l) for l in range(case["layers"])], L_p=case["L_p"],
                                     L_r=case["L_r"], rho=case["rho"], K_p=K_p, K_r=K_r, rms_eps=EPS, rope_theta=THETA,
                                     paging=paging)
        first, second, _ = _hiddens(case, seed)
        state = {"op": op, "mode": case["mode"], "den": den, "first": first, "second": second, "i": 1}
        if case["mode"] != "full":
            den.step(first, 0)  # the caches a running generation has
        return state
    if op == "head":
        hidden, gain, lm, rows = _head_inputs(case, seed)
        return {"op": op, "hidden": hidden, "gain": gain, "lm": lm, "rows": rows}
    if op == "attention":
        q, k, v = _attention_inputs(case, seed)
        return {"op": op, "q": q, "k": k, "v": v, "case": case}
    if op == "linear":
        a, w, rows = _linear_inputs(case, seed)
        return {"op": op, "a": a, "w": w, "rows": rows, "dtype": case["dtype"]}
    if op == "vverify":
        first, second, wv = _vverify_inputs(case, seed)
        cache = (first.float() @ wv.float().t()).to(torch.bfloat16)
        return {"op": op, "first": first, "second": second, "wv": wv, "cache": cache}
    return {"op": op, "scores": _scores(case, seed), "k": case["k"]}


def run(state):
    op = state["op"]
    if op == "step":
        den, mode = state["den"], state["mode"]
        if mode == "full":
            return den.step(state["second"], 0)[0]
        if mode == "response":
            out, _ = den.step(state["second"], state["i"])
            state["i"] += 1
            return out
        # the changed tokens arrive, and change back
        out2, n_sel = den.step(state["second"], state["i"])
        out1, _ = den.step(state["first"], state["i"] + 1)
        state["i"] += 2
        return {"second": out2, "first": out1, "selected": den.sel_idx[:, :, :n_sel]}
    if op == "head":
        x0, conf = binding.op_head("bf16", state["hidden"], state["gain"], state["lm"], EPS, rows=state["rows"])
        return {"token": x0, "confidence": conf}
    if op == "attention":
        c = state["case"]
        return binding.op_attention(c["dtype"], state["q"], state["k"], state["v"], c["H_q"], c["H_kv"], c["d_h"])
    if op == "linear":
        return binding.op_linear(state["dtype"], state["a"], state["w"], row_idx=state["rows"])
    if op == "vverify":
        s2 = binding.op_vverify("bf16", state["second"], state["wv"], state["cache"])
        s1 = binding.op_vverify("bf16", state["first"], state["wv"], state["cache"])
        return {"second": s2, "first": s1, "cache": state["cache"]}
    return binding.op_select(state["scores"], state["k"])


# ---------------------------------------------------------------------------------------- work, tolerance

def work(case):
    op = case["op"]
    esz = 4 if case.get("dtype") == "f32" else 2
    if op == "step":
        H_q, H_kv, d_h, d, m, _ = MODELS[case["model"]]
        d_q, d_kv = H_q * d_h, H_kv * d_h
        B, L_p, L_r = case["B"], case["L_p"], case["L_r"]
        n = L_p + L_r
        P = case["mode"] in ("full", "prompt")
        carried = B * (n if P else L_r)
        again = B * ((L_p if P else 0) + (L_r if case["mode"] in ("full", "response") else _k(case)))
        weights = d * d_q + 2 * d * d_kv + d_q * d + 3 * d * m
        flops = 2.0 * carried * d * d_kv + 2.0 * again * (d * d_q + d * d_kv + d_q * d + 3 * d * m) + 4.0 * again * n * d_q
        # weights once; cached keys and values read or, where new, written; cached outputs of the carried rows
        # read or written
        nbytes = esz * (weights + 2 * B * n * d_kv + 2 * carried * d)
        steps = 1 if case["mode"] in ("full", "response") else 2
        io = esz * (carried * d + B * n * d)
        return {"bytes": steps * (case["layers"] * nbytes + io), "flops": steps * case["layers"] * flops}
    if op == "head":
        d, vocab = MODELS[case["model"]][3], MODELS[case["model"]][5]
        return {"bytes": 2.0 * vocab * d + 2.0 * case["M"] * d + 8.0 * case["M"], "flops": 2.0 * case["M"] * vocab * d}
    if op == "attention":
        B, Mq, n, d_q, d_kv = case["B"], case["Mq"], case["n"], case["H_q"] * case["d_h"], case["H_kv"] * case["d_h"]
        return {"bytes": esz * B * (2.0 * Mq * d_q + 2.0 * n * d_kv), "flops": 4.0 * B * Mq * n * d_q}
    if op == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": esz * (N * K + M * K) + 4.0 * M * N, "flops": 2.0 * M * N * K}
    if op == "vverify":
        H_q, H_kv, d_h, d, _, _ = MODELS[case["model"]]
        r, d_kv = case["rows"], H_kv * d_h
        return {"bytes": 2 * (2.0 * d * d_kv + 2.0 * r * d + 4.0 * r * d_kv + 4.0 * r), "flops": 2 * 2.0 * r * d * d_kv}
    return {"bytes": 4.0 * case["B"] * (case["L"] + case["k"]), "flops": 0.0}


def _cost(case):
    """Seconds, roughly: what bounds draw()."""
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / (8e12 if case.get("dtype") == "f32" else 8e14)


def tolerance(case):
    """Measured by running the same inputs through other kernels and contraction splits of the library and against
    exact(), times about four: bf16 steps moved by up to 4.6e-3 (largest element 2.8e-2), float32 steps are up to
    6e-7 from their 64-bit values, float32 results of a linear map moved by 4e-7 (3e-6), confidences of bf16 rows
    are 7e-4 from theirs; a bf16 result of attention is 1.7e-3 away by its last rounding alone."""
    op = case["op"]
    if op == "select":
        return "exact"
    if op == "step":
        return {"rel": 4e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.1}
    if op == "head":
        return {"rel": 3e-3, "max": 1e-2, "differ": 0.01}
    if op == "linear":
        return {"rel": 4e-6, "max": 4e-5}
    if op == "attention":
        return {"rel": 3e-3, "max": 2e-2}
    return {"rel": 3e-3, "max": 2e-2}


# ---------------------------------------------------------------------------------------- 64-bit values

def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * gain


def _rope(x, pos, d_h):
    """x [..., rows, heads * d_h] at positions pos [..., rows]."""
    half = d_h // 2
    w = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / d_h)
    ang = pos.to(torch.float64)[..., None, None] * w
    y = x.reshape(*x.shape[:-1], -1, d_h)
    a, b = y[..., :half], y[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], dim=-1).reshape(x.shape)


def _attend(q, k, v, H_q, H_kv, d_h):
    """[rows, H_q * d_h] against [n, H_kv * d_h], one sequence."""
    out = torch.empty_like(q)
    for a in range(H_q):
        kv = a // (H_q // H_kv)
        s = q[:, a * d_h:(a + 1) * d_h] @ k[:, kv * d_h:(kv + 1) * d_h].t() / math.sqrt(d_h)
        out[:, a * d_h:(a + 1) * d_h] = torch.softmax(s, dim=-1) @ v[:, kv * d_h:(kv + 1) * d_h]
    return out


class _Model64:
    """The cached step in 64 bits: caches of every layer, and which rows a step carries and recomputes."""

    def __init__(self, case, seed):
        self.case = case
        self.layers = [{k: t.double() for k, t in _layer(case, seed, l).items()} for l in range(case["layers"])]
        self.caches = [{} for _ in self.layers]

    def step(self, hidden, first_carried, again):
        """again [B, r]: positions recomputed, among the carried ones first_carried .. n-1."""
        H_q, H_kv, d_h, d, m, _ = MODELS[self.case["model"]]
        x = hidden.double()[:, first_carried:].clone()
        B = x.shape[0]

        def rows(t, width):
            return (again - first_carried)[:, :, None].expand(B, again.shape[1], width)

        def put(c, name, val, n_rows):
            if name not in c:
                c[name] = torch.zeros((B, n_rows, val.shape[-1]), dtype=torch.float64, device=val.device)
            c[name] = c[name].scatter(1, again[:, :, None].expand(B, again.shape[1], val.shape[-1]), val)

        for w, c in zip(self.layers, self.caches):
            n = hidden.shape[1]
            h = _rms(x, w["attn_norm_g"])
            v = h @ w["wv"].t()
            c["v"] = v if first_carried == 0 else torch.cat([c["v"][:, :first_carried], v], dim=1)
            hr = h.gather(1, rows(h, d))
            q = _rope(hr @ w["wq"].t(), again, d_h)
            put(c, "k", _rope(hr @ w["wk"].t(), again, d_h), n)
            o = torch.stack([_attend(q[b], c["k"][b], c["v"][b], H_q, H_kv, d_h) for b in range(B)])
            put(c, "ao", o @ w["wo"].t(), n)
            x = x + c["ao"][:, first_carried:]
            f = _rms(x.gather(1, rows(x, d)), w["ffn_norm_g"])
            u = torch.nn.functional.silu(f @ w["w_gate"].t()) * (f @ w["w_up"].t())
            put(c, "fo", u @ w["w_down"].t(), n)
            x = x + c["fo"][:, first_carried:]
        if first_carried == 0:
            self.prompt_out = x[:, :self.case["L_p"]]
            return x
        return torch.cat([self.prompt_out, x], dim=1)


def exact(case, seed):
    op = case["op"]
    if op == "step":
        B, L_p, L_r = case["B"], case["L_p"], case["L_r"]
        n = L_p + L_r
        first, second, changed = _hiddens(case, seed)
        m = _Model64(case, seed)
        every = torch.arange(n, device="cuda").expand(B, n)
        if case["mode"] == "full":
            return m.step(second, 0, every)
        m.step(first, 0, every)
        if case["mode"] == "response":
            return m.step(second, L_p, every[:, L_p:])
        if case["mode"] == "prompt":
            start, again = 0, torch.cat([every[:, :L_p], changed], dim=1)
        else:
            start, again = L_p, changed
        return {"second": m.step(second, start, again), "first": m.step(first, start, again), "selected": None}
    if op == "head":
        hidden, gain, lm, rows = _head_inputs(case, seed)
        logits = _rms(hidden[rows.long()].double(), gain.double()) @ lm.double().t()
        return {"token": None, "confidence": torch.softmax(logits, dim=-1).max(dim=-1).values}
    if op == "attention":
        q, k, v = _attention_inputs(case, seed)
        return torch.stack([_attend(q[b].double(), k[b].double(), v[b].double(), case["H_q"], case["H_kv"], case["d_h"])
                            for b in range(case["B"])])
    if op == "linear":
        a, w, rows = _linear_inputs(case, seed)
        return a[rows.long()].double() @ w.double().t()
    if op == "vverify":
        first, second, wv = _vverify_inputs(case, seed)
        v1, v2 = first.double() @ wv.double().t(), second.double() @ wv.double().t()
        cos = torch.nn.functional.cosine_similarity(v1, v2, dim=-1)
        return {"second": cos, "first": cos, "cache": v1}
    return None
