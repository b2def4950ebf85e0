// Gathered linear maps of float32 models,  C[i, :] = A[rows[i], :] * W^T, on the float32 matrix
// instructions (v_mfma_f32_16x16x4_f32: products and sums in float32, 157 TFLOP/s on the chip).
//
// An instruction multiplies four values of the contraction index in 32 cycles, 16 times the cycles per
// byte of the bf16 instructions: what bounds these launches is the chain of instructions of the busiest
// wavefront, and below some 0.1 GFLOP a trip to memory.
//
// k_gemm_f32<MI, NJ, KW, PAIR>: a 16*MI x 16*NJ tile per workgroup, KW wavefronts that each take a part
// of its contraction range, no LDS on the way in: every lane reads 16 bytes of its row (row lane % 16 of a
// block, contraction values 4 * (lane / 16) .. + 3 of a chunk of 16) straight into the registers that
// feed four instructions, four chunks ahead.  Four short chains instead of one long one: the kernel for few rows
// and for small maps.
// k_gemm_f32_lds: 64 x 64 tiles through LDS, for the others.
// Against the plain LDS kernel that float32 models used (k_gemm_simple: vector FMAs, one 64 x 64 tile per
// workgroup, no slices), op_linear with its slice sum, us: 8 x 256 x 256 36 -> 7; 32 x 256 x 704 91 -> 8;
// 40 x 1024 x 3072 385 -> 11; 352 x 1024 x 1024 134 -> 17; 352 x 6144 x 1024 170 -> 57 (77 TFLOP/s);
// 64 x 4096 x 4096 600 -> 27; 2048 x 4096 x 4096 1477 -> 580 (118 TFLOP/s; the library's product of
// 4096^3 134).
#include <type_traits>

#include "common.hpp"

namespace dllmc {

namespace {

template <int MI, int NJ, int KW, int PAIR>
__global__ __launch_bounds__(64 * KW, 2) void k_gemm_f32(
    const float* __restrict__ A, int lda, const int* __restrict__ rows, int M,
    const float* __restrict__ W0, const float* __restrict__ W1, int N0, int N, int K,
    int k_per_slice, float* __restrict__ C, float* __restrict__ U) {
  constexpr int WC = PAIR ? NJ / 2 : NJ;  // column blocks of the output
  constexpr int PF = 4;                   // chunks in flight
  static_assert(!PAIR || NJ % 2 == 0, "gate and up column blocks come in pairs");
  const int kw = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  int col_tile, row_tile;
  xcd_tile_map_blocked(col_tile, row_tile);
  const int m0 = row_tile * 16 * MI, n0 = col_tile * 16 * WC;

  // this wavefront's chunks [c0, c1) of 16 contraction values, of the workgroup's slice
  const int kbeg = blockIdx.z * k_per_slice, kend = min(K, kbeg + k_per_slice);
  const int nch_all = (kend - kbeg + 15) / 16;
  const int per = (nch_all + KW - 1) / KW;
  const int c0 = min(kw * per, nch_all), c1 = min(nch_all, c0 + per);
  const int nch = c1 - c0;

  // rows and columns past the end repeat the last one and are dropped at the store
  const float* ap[MI];
  const float* bp[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = min(m0 + i * 16 + ln, M - 1);
    ap[i] = A + static_cast<size_t>(rows ? rows[m] : m) * lda;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = min(n0 + (j % WC) * 16 + ln, N - 1);
    if (PAIR) bp[j] = (j < WC ? W0 : W1) + static_cast<size_t>(n) * K;
    else bp[j] = n < N0 ? W0 + static_cast<size_t>(n) * K : W1 + static_cast<size_t>(n - N0) * K;
  }

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  f32x4 a[PF][MI], b[PF][NJ];
  // (a chunk past the range, or a lane's four values past K, re-read the row's last four values; the
  // former are never multiplied, the latter zeroed first)
  auto load = [&](int u, int c) {
    const int k = min(kbeg + (c0 + c) * 16 + lg * 4, K - 4);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[u][i] = *reinterpret_cast<const f32x4*>(ap[i] + k);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[u][j] = *reinterpret_cast<const f32x4*>(bp[j] + k);
  };
  auto multiply = [&](int u) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][t], b[u][j][t], acc[i][j], 0, 0, 0);
  };
  if (nch > 0) {
#pragma unroll
    for (int u = 0; u < PF; ++u) load(u, u);
    int base = 0;
    for (; base + PF < nch; base += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        multiply(u);
        load(u, base + u + PF);
        __builtin_amdgcn_sched_barrier(0);  // (the compiler would sink the loads to their use)
      }
    }
    // the last 1 .. PF chunks: the only ones that can hold values past the slice (K % 16)
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (base + u < nch) {
        const bool in = kbeg + (c0 + base + u) * 16 + lg * 4 < kend;
#pragma unroll
        for (int i = 0; i < MI; ++i)
          if (!in) a[u][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          if (!in) b[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        multiply(u);
      }
  }

  if (KW > 1) {
    // the groups' sums meet in LDS and are added in group order by the first one
    __shared__ f32x4 red[(KW - 1) * MI * NJ * 64];
    if (kw > 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          red[((kw - 1) * MI * NJ + i * NJ + j) * 64 + lane] = acc[i][j];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll
    for (int g = 1; g < KW; ++g)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] += red[((g - 1) * MI * NJ + i * NJ + j) * 64 + lane];
  }

  float* Cs = PAIR ? U : C + static_cast<size_t>(blockIdx.z) * M * N;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + i * 16 + lg * 4 + e;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < WC; ++j) {
        const int n = n0 + j * 16 + ln;
        if (n >= N) continue;
        float v = acc[i][j][e];
        if (PAIR) v = v / (1.0f + expf(-v)) * acc[i][j + NJ - WC][e];
        Cs[static_cast<size_t>(m) * N + n] = v;
      }
    }
}

// k_gemm_f32_lds<MI, NJ, PAIR>: 2 x 2 wavefronts of 16*MI rows x 16*NJ columns, operands through LDS
// (global_load_lds_dwordx4: an instruction copies 8 rows x 128 bytes = 32 contraction values; slot of
// chunk c of row r is c ^ (r % 8), so that the fragment reads of 8 rows hit 8 bank groups) in a ring
// of three stages of 32 contraction values.
// The register kernel above stops at 75 TFLOP/s however many workgroups it has (its loads touch 16 rows per
// instruction; a CU took them at ~16 bytes per cycle, with or without sharing in the L1).  Here the loads are
// whole 128-byte lines and every byte serves two wavefronts: 118 TFLOP/s.  128 x 128 tiles (64 x 64 per
// wavefront, two stages) gained 3 % above 768 rows and lost below; 64 x 128 lay between.
// (The body is a function of its own, inlined: with the loads issued from the kernel itself the compiler
// waits for every load in flight before each LDS read.)
template <int MI, int NJ, int PAIR>
__device__ __forceinline__ void gemm_f32_lds_body(
    const float* __restrict__ A, int lda, const int* __restrict__ rows, int M,
    const float* __restrict__ W0, const float* __restrict__ W1, int N0, int N, int K,
    int k_per_slice, float* __restrict__ C, float* __restrict__ U) {
  constexpr int BM = 32 * MI, BW = 32 * NJ;        // tile rows, weight rows of the tile
  constexpr int BN = PAIR ? BW / 2 : BW;           // output columns
  constexpr int LA = BM / 32, LB = BW / 32;        // load instructions per wavefront and stage
  constexpr int NST = 3;
  constexpr int kStage = (BM + BW) * 8;
  __shared__ __attribute__((aligned(1024))) uint4 lds[NST][kStage];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  const int wm = wave / 2, wn = wave % 2;
  int col_tile, row_tile;
  xcd_tile_map_blocked(col_tile, row_tile);
  const int m0 = row_tile * BM, n0 = col_tile * BN;
  const int kbeg = blockIdx.z * k_per_slice, kend = min(K, kbeg + k_per_slice);
  const int nkt = (kend - kbeg + 31) / 32;

  // loader: instruction q covers tile rows [8q, 8q + 8); lane l: row 8q + l/8, slot l%8, chunk
  // (l%8) ^ (row%8).  Rows past the end repeat the last one.
  const float* asrc[LA];
  const float* bsrc[LB];
  const int chunk = (lane % 8) ^ (lane / 8);  // 8q % 8 == 0
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int m = min(m0 + 8 * (LA * wave + j) + lane / 8, M - 1);
    asrc[j] = A + static_cast<size_t>(rows ? rows[m] : m) * lda;
  }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int r = 8 * (LB * wave + j) + lane / 8;
    if (PAIR) {
      const int n = min(n0 + r % BN, N - 1);
      bsrc[j] = (r < BN ? W0 : W1) + static_cast<size_t>(n) * K;
    } else {
      const int n = min(n0 + r, N - 1);
      bsrc[j] = n < N0 ? W0 + static_cast<size_t>(n) * K : W1 + static_cast<size_t>(n - N0) * K;
    }
  }
  auto issue = [&](int stage, int kt) {
    // (values past K: any that are there; the last step zeroes them)
    const int k = min(kbeg + kt * 32 + chunk * 4, K - 4);
#pragma unroll
    for (int j = 0; j < LA; ++j)
      __builtin_amdgcn_global_load_lds(asrc[j] + k, &lds[stage][(LA * wave + j) * 64], 16, 0, 0);
#pragma unroll
    for (int j = 0; j < LB; ++j)
      __builtin_amdgcn_global_load_lds(bsrc[j] + k, &lds[stage][BM * 8 + (LB * wave + j) * 64], 16, 0, 0);
  };

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto step = [&](auto last_tag, int kt, int stage) {
    constexpr bool LAST = decltype(last_tag)::value;
    const uint4* la = &lds[stage][0];
    const uint4* lb = &lds[stage][BM * 8];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int c = kk * 4 + lg;
      f32x4 a[MI], b[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = wm * (MI * 16) + i * 16 + ln;
        a[i] = __builtin_bit_cast(f32x4, la[r * 8 + (c ^ (r % 8))]);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int r = PAIR ? (j / (NJ / 2)) * BN + wn * (NJ / 2 * 16) + (j % (NJ / 2)) * 16 + ln
                           : wn * (NJ * 16) + j * 16 + ln;
        b[j] = __builtin_bit_cast(f32x4, lb[r * 8 + (c ^ (r % 8))]);
      }
      if (LAST && kbeg + kt * 32 + c * 4 >= kend) {
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
    }
  };
  // this wavefront's loads of step kt have landed and its fragment reads of step kt - 1 are complete;
  // behind the barrier that holds for everybody, and the stage of step kt - 1 is free
#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nkt) issue(s, s);
  for (int kt = 0; kt + 1 < nkt; ++kt) {
    wait_vmcnt_lds<LA + LB>();  // the step after it may be in flight
    __builtin_amdgcn_s_barrier();
    if (kt + NST - 1 < nkt) issue((kt + NST - 1) % NST, kt + NST - 1);
    step(std::integral_constant<bool, false>{}, kt, kt % NST);
  }
  wait_vmcnt_lds<0>();
  __builtin_amdgcn_s_barrier();
  step(std::integral_constant<bool, true>{}, nkt - 1, (nkt - 1) % NST);

  float* Cs = PAIR ? U : C + static_cast<size_t>(blockIdx.z) * M * N;
  constexpr int WC = PAIR ? NJ / 2 : NJ;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + wm * (MI * 16) + i * 16 + lg * 4 + e;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < WC; ++j) {
        const int n = n0 + wn * (WC * 16) + j * 16 + ln;
        if (n >= N) continue;
        float v = acc[i][j][e];
        if (PAIR) v = v / (1.0f + expf(-v)) * acc[i][j + NJ - WC][e];
        Cs[static_cast<size_t>(m) * N + n] = v;
      }
    }
}

template <int MI, int NJ, int PAIR>
__global__ __launch_bounds__(256, 2) void k_gemm_f32_lds(
    const float* __restrict__ A, int lda, const int* __restrict__ rows, int M,
    const float* __restrict__ W0, const float* __restrict__ W1, int N0, int N, int K,
    int k_per_slice, float* __restrict__ C, float* __restrict__ U) {
  gemm_f32_lds_body<MI, NJ, PAIR>(A, lda, rows, M, W0, W1, N0, N, K, k_per_slice, C, U);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// tile shapes: rows, columns (weight rows), groups over the contraction range, measured time over the
// time of the instruction chains
struct Shape { int bm, bn, kw; double slow; };
constexpr Shape kShapes[2] = {{32, 32, 4, 2.1}, {64, 64, 1, 1.4}};

}  // namespace

bool gemm_f32_ok(const void* A, int lda, const void* W0, const void* W1, int K) {
  return K % 4 == 0 && lda % 4 == 0 && aligned16(A) && aligned16(W0) && (W1 == nullptr || aligned16(W1));
}

// Estimated time in us of both kernels at every slice count; the cheapest is taken.  2 us for the trip
// to memory that every launch makes, rounds of workgroups over the 256 CUs (a CU's four SIMDs take a
// wavefront each, so the workgroups that share a CU take turns) times a wavefront's instructions (16 per
// 16 contraction values, 32 cycles each) times the kernel's measured factor, and the partial sums,
// which mostly stay in the memory-side cache.  Slices are whole 256-byte pieces of a row (at a multiple of
// 64 bytes a launch takes a fifth longer).  Within 10 % of the best measured choice over 30 shapes from
// 8 x 256 x 256 to 2048 x 4096 x 4096.
F32Plan plan_f32(int M, int N, int K, int s_cap, int force_s) {
  F32Plan best{};
  best.t = 1e30;
  for (int sh = 0; sh < 2; ++sh) {
    const Shape& s = kShapes[sh];
    const int mt = (M + s.bm - 1) / s.bm, nt = (N + s.bn - 1) / s.bn;
    const int s_hi = force_s > 0 ? (force_s < s_cap ? force_s : s_cap) : s_cap;
    for (int S = force_s > 0 ? s_hi : 1; S <= s_hi; ++S) {
      int kps = ((K + S - 1) / S + 63) / 64 * 64;
      if (kps > K) kps = K;
      const int used = (K + kps - 1) / kps;
      const double rounds = static_cast<double>((static_cast<long long>(mt) * nt * used + 255) / 256);
      const int chunks = ((kps + 15) / 16 + s.kw - 1) / s.kw;
      const double t_part = used > 1 ? used * (2.0 * M * N * 4.0 / 8e6 + 0.15) : 0.0;
      const double t = 2.0 + rounds * chunks * 16.0 * 32.0 / 2400.0 * s.slow + t_part;
      if (t < best.t * 0.98) best = F32Plan{sh, used, kps, nt, mt, t};
    }
  }
  return best;
}

void launch_gemm_f32(const F32Plan& p, const float* A, int lda, const int* rows, int M, const float* W0,
                     const float* W1, int N0, int N, int K, float* C, hipStream_t st) {
  const dim3 grid(p.nt, p.mt, p.S);
#define DLLMC_F32(KERNEL) \
  hipLaunchKernelGGL(KERNEL, grid, dim3(256), 0, st, A, lda, rows, M, W0, W1, N0, N, K, p.kps, C, nullptr)
  if (p.shape == 0) DLLMC_F32((k_gemm_f32<2, 2, 4, 0>));
  else DLLMC_F32((k_gemm_f32_lds<2, 2, 0>));
#undef DLLMC_F32
}

bool launch_gemm_f32_swiglu(const float* A, int lda, const int* rows, int M, const float* w_gate,
                            const float* w_up, int m, int K, float* u, hipStream_t st) {
  // Gate and up together in one slice, finished in the tile (its columns are half gate, half up) --
  // unless slices and a second launch (4 us, and the sums once more through memory) are quicker: few
  // rows against a long contraction.
  const F32Plan p = plan_f32(M, 2 * m, K, 1, 0), split = plan_f32(M, 2 * m, K, kMaxSlices, 0);
  if (p.t > split.t + 4.0 + 2.0 * M * 2.0 * m * 4.0 / 8e6) return false;
#define DLLMC_F32(KERNEL, BN)                                                                       \
  hipLaunchKernelGGL(KERNEL, dim3((m + BN - 1) / BN, p.mt, 1), dim3(256), 0, st, A, lda, rows, M, w_gate, \
                     w_up, m, m, K, K, nullptr, u)
  if (p.shape == 0) DLLMC_F32((k_gemm_f32<2, 2, 4, 1>), 16);
  else DLLMC_F32((k_gemm_f32_lds<2, 2, 1>), 32);
#undef DLLMC_F32
  return true;
}

}  // namespace dllmc
