"""Host-side logic of the library that needs no GPU: the GEMM slice planner never plans more
float32 partial sums than the slice buffer holds (an overflow there is an out-of-bounds write
on the device), for every shape the workloads produce and for random ones."""
import ctypes
import os

import numpy as np
import pytest

from paper_2506_06295_amd import binding, inputs as I

pytestmark = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="libdllmc.so not built")


def workspace_cws_floats(cfg):
    # mirrors make_layout(): rows padded to 128 times the widest GEMM output, plus 640 tiles
    rows = cfg.B * cfg.n
    n_max = max(2 * cfg.m, cfg.d_q + cfg.d_kv, cfg.d)
    return (rows + 127) // 128 * 128 * n_max + 640 * 128 * 128


def step_gemm_shapes(cfg):
    k = int(np.floor(cfg.rho * cfg.L_r + 1e-6))
    for P in (False, True):
        for Rf in (False, True):
            Mc = cfg.B * ((cfg.L_p if P else 0) + cfg.L_r)
            M_R = cfg.B * ((cfg.L_p if P else 0) + (cfg.L_r if Rf else k))
            yield Mc, cfg.d_kv, cfg.d_kv, cfg.d
            if M_R:
                yield M_R, cfg.d_q + cfg.d_kv, cfg.d_q, cfg.d
                yield M_R, cfg.d, cfg.d, cfg.d_q
                yield M_R, 2 * cfg.m, cfg.m, cfg.d
                yield M_R, cfg.d, cfg.d, cfg.m


@pytest.mark.parametrize("name", list(I.CONFIGS))
def test_planned_slices_fit_the_workspace_for_every_step_kind(name):
    cfg = I.CONFIGS[name]
    L = binding.lib()
    cap = workspace_cws_floats(cfg)
    dt = 1 if cfg.dtype == "bf16" else 0
    for rho in (cfg.rho, 0.05, 0.5, 1.0):
        c = cfg.replace(rho=rho)
        for M, N, N0, K in step_gemm_shapes(c):
            S = L.dllmc_plan_gemm_slices(dt, M, N, N0, K, cap)
            assert 1 <= S <= 8, (M, N, K, S)
            assert S * M * N <= cap, (M, N, K, S)


def test_planned_slices_respect_any_capacity():
    L = binding.lib()
    r = np.random.default_rng(0)
    for _ in range(3000):
        M = int(r.integers(1, 20000))
        N = int(r.choice([128, 256, 512, 1024, 4096, 8192, 24576, 37888, 200, 704]))
        K = int(r.choice([128, 256, 512, 896, 1024, 3584, 4096, 12288, 18944, 72]))
        cap = int(r.integers(1, 9)) * M * N + int(r.integers(0, 1000)) - (M * N if r.random() < 0.1 else 0)
        for dt in (0, 1):
            S = L.dllmc_plan_gemm_slices(dt, M, N, N, K, max(cap, 0))
            if cap < M * N:
                assert S == 0
            else:
                assert S >= 1 and S * M * N <= cap


def test_bench_refuses_more_than_one_gpu():
    """bench.py runs on one GPU; asking for more ends with a message, before anything touches a GPU."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def test_attention_of_few_queries_plan():
    """Kernel and key ranges by estimated time: many workgroups on short sequences walk their keys together (the kernel
    whose wavefronts split them starts anew with every round over the CUs); few of them split, as scratch allows."""
    L = binding.lib()

    def plan(B, Mq, n, H_q, H_kv, split=1):
        queries = ctypes.c_int32(99)
        ranges = L.dllmc_plan_attention(B, Mq, n, H_q, H_kv, split, ctypes.byref(queries))
        return queries.value, ranges

    for B, Mq, n, H_q, H_kv in [(16, 100, 100, 28, 4), (16, 127, 250, 32, 32), (8, 51, 300, 32, 32), (8, 65, 100, 28, 4),
                                (8, 33, 100, 32, 32)]:
        assert plan(B, Mq, n, H_q, H_kv) == (0, 1), (B, Mq, n)
    assert plan(1, 51, 4608, 32, 32) == (32, 4)
    assert plan(1, 51, 4608, 32, 32, split=0)[1] == 1
    for B in (1, 3, 8):
        for Mq in (1, 17, 64, 127):
            for n in (1, 33, 700, 5000):
                q0, r0 = plan(B, Mq, n, 28, 4)
                per = {-1: 64, 0: 64}.get(q0, q0)
                assert 1 <= r0 <= 16 and (r0 == 1 or B * -(-Mq // per) * 28 * r0 <= 256)
                assert q0 != -1 or -(-(-(-n // 32)) // r0) <= 3  # ranges that are fetched at once
    assert L.dllmc_plan_attention(1, 128, 100, 4, 4, 1, None) < 0
    assert L.dllmc_plan_attention(1, 8, 100, 4, 3, 1, None) < 0


def test_vverify_plan():
    """By estimated time: one round of 64 x 64 tiles, the larger tiles where they fill their rounds, else the split
    contraction (in the gaps between whole rounds it is ahead at every width)."""
    plan = binding.lib().dllmc_plan_vverify
    for rows, d, d_kv, way in [(64, 4096, 4096, 0), (256, 4096, 4096, 4), (448, 4096, 4096, 0), (576, 4096, 4096, 0),
                               (768, 4096, 4096, 0), (900, 4096, 4096, 0), (1280, 4096, 4096, 0), (1280, 8192, 8192, 0),
                               (2048, 4096, 4096, 1), (4096, 4096, 4096, 2), (1000, 2560, 2560, 3), (1280, 3584, 512, 4)]:
        assert plan(1, rows, d, d_kv) == way, (rows, d, d_kv)
    assert plan(0, 256, 4096, 4096) == 0            # float32
    assert plan(1, 256, 4096, 4100) == 0            # columns that 64 does not divide
    assert plan(1, 256, 4100, 4096) == 0            # nor the contraction
    assert plan(1, 0, 64, 64) < 0 and plan(2, 1, 64, 64) < 0


def test_vverify_plan_takes_the_quicker_way():
    """Sizes at which the way taken once was not the quicker of those timed (us): 58.7 in 256 x 256 tiles against 46.2 in 192 x
    256, 73.2 against 57.8, 42.5 against 34.6, 42.2 in 64 x 64 against 30.6 in 192 x 64; and two that estimates of another form lost (64 x 64 tiles 13.4 against 14.6, 8.6 against 9.4)."""
    plan = binding.lib().dllmc_plan_vverify
    for rows, d, d_kv, way in [(4608, 2048, 2048, 3), (3300, 2560, 2560, 3), (12288, 1024, 1024, 3), (4096, 3584, 512, 3),
                               (192, 2048, 2048, 4), (333, 896, 128, 4)]:
        assert plan(1, rows, d, d_kv) == way, (rows, d, d_kv)
