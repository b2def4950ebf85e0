// Gathered linear maps of few rows (an adaptive step's recomputed rows) against a weight matrix that is
// read once, bf16; also the general kernel for column counts that the 128 / 256-column tiles do not divide.
//
// k_gemm_ring<RB, NB, DUAL>: tile = 64 * RB rows x 16 * NB weight rows, one workgroup of eight wavefronts per
// CU.  Both operands go from global memory straight into LDS (global_load_lds_dwordx4: an instruction
// copies 8 rows x 128 bytes), through a ring of as many 64-wide stages as 150 KB hold, at most eight.  All but one
// of them are in flight per CU, seven steps of the smallest tiles (56 KB of weights at NB = 4), two of the largest (32 to 40
// KB at RB = 3, NB = 8 and 10), and not drained before the last steps.  Four wavefronts
// take 16 * RB rows each for the first half of every step, the other four the same rows for its second half
// (so that any number of column blocks deals evenly); their sums meet in LDS at the end.
//   DUAL = 1: NB/2 blocks of W0 (gate) and the same blocks of W1 (up); the epilogue stores
//             bf16(silu(gate) * up) to U[M, N].  One slice.
//   FINE: the float32 sums are the caller's result, not what a row kernel rounds: fewer slices mean longer chains of
//             additions, so the steps are dealt to two or four sums per element, at 0.1 to 0.4 us (error against 64 bits, one
//             slice of 333 x 3072 x 1024: 1.28e-7 -> 7.7e-8; two of 333 x 4096 x 4096: 1.69e-7 -> 1.23e-7).
//   NT: non-temporal weight loads, for weights that only one workgroup reads and that no cache will hold when they are
//             read again (launches of one row tile in models whose weights exceed the 256 MB memory-side cache): they then displace
//             neither what the launch's workgroups share nor what the next launches read, and come at 6.0 TB/s
//             instead of 5.3 (a loop of nothing but these loads, 201 MB of weights beside 64 activation rows: 37.8 -> 33.7 us).
//             Layer of an adaptive step of 64 rows, 4096 wide: gate/up 45.5 -> 38.6 us, down 29.8 -> 25.9, Q|K 20.8 -> 19.2, and
//             the launches between them 3 us less; of 62 rows, 3584 wide: 57.7 -> 50.2, 34.6 -> 30.8.
//   otherwise columns [0, N0) come from W0, [N0, N) from W1, float32 partial sums of slice blockIdx.z go
//             to C[z]; the row kernels add the slices in order (no float atomics: bit-reproducible).
// Columns past N and rows past M repeat the last one and are dropped at the store: any M and N.
//
// Bound by the weight stream: launches take about 4 us + bytes / 5.5 TB/s.  Measured on weights that no cache holds, us, with the kernel
// before (weight rows straight into the MFMA operand, 16 rows x 64 bytes per load instruction, which
// a CU takes at half the rate of whole lines; activations through registers into LDS):
//   64 rows:  4096 x 4096 10.9 -> 10.1 (and 4 slices instead of 8), 8192 x 4096 17.8 -> 16.3 (2 instead of 4),
//             4096 x 12288 23.2 -> 23.1 (4 instead of 8), 3584 x 18944 33.8 -> 27.7,
//             gate/up 2 x 12288 x 4096 43.9 -> 38.4, 2 x 18944 x 3584 71.7 -> 51.0
//   128 rows: 4096 x 4096 14.8 -> 12.6, 8192 x 4096 22.3 -> 19.3, gate/up 59.4 -> 44.9 and 101 -> 59
//   160 rows: 18.7 -> 15.3, 29.9 -> 23.9, 4096 x 12288 41.7 -> 30.4
// From 192 rows the 128 x 128 tiles are level or ahead in many places (256 rows: 16.9 / 27.2 / 39.3 us there, 17.4 / 26.8 /
// 36.6 here; gate/up 62 there, 68 here), and plan_gemm takes the one with the lower estimate.
#include <type_traits>

#include "common.hpp"

namespace dllmc {

namespace {

// (The body is a function of its own, inlined: with the loads issued from the kernel itself the compiler
// waits for every load in flight before each LDS read.)
template <int RB, int NB, int DUAL, bool FINE, bool NT>
__device__ __forceinline__ void gemm_ring_body(const bf16_t* __restrict__ A, int lda,
                                               const int* __restrict__ rows, int M,
                                               const bf16_t* __restrict__ W0,
                                               const bf16_t* __restrict__ W1, int N0, int N, int K,
                                               int k_per_slice, float* __restrict__ C,
                                               bf16_t* __restrict__ U) {
  constexpr int BM = 64 * RB;
  constexpr int CB = DUAL ? NB / 2 : NB;               // column blocks of the output
  constexpr int kStage = (BM + 16 * NB) * 8;           // 16-byte slots
  constexpr int kFit = (150 * 1024) / (kStage * 16);
  constexpr int NST = kFit > 8 ? 8 : kFit;
  constexpr int LA = RB, LBT = 2 * NB;                 // activation loads per wavefront; weight loads of all
  constexpr int LB0 = LBT / 8, LBR = LBT % 8;          // ... per wavefront, one more for the first LBR
  constexpr int kAux = NT ? 2 : 0;                     // non-temporal weight loads
  // FINE: sums of the steps kt % NA = 0, 1, ... apart, NA shorter chains of additions that are added up at the end
  constexpr int NA = !FINE ? 1 : RB * NB <= 12 ? 4 : 2;
  __shared__ __attribute__((aligned(1024))) uint4 lds[NST][kStage];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  const int wr = wave % 4, kk = wave / 4;
  int col_tile, row_tile;
  xcd_tile_map(col_tile, row_tile);
  const int m0 = row_tile * BM, cb0 = col_tile * CB;
  const int kbeg = blockIdx.z * k_per_slice;
  const int klen = min(K, kbeg + k_per_slice) - kbeg;  // multiple of 64
  const int nkt = klen / 64;

  // loader: an instruction copies 8 rows x 128 bytes; lane l: row 8q + l/8, slot l%8, chunk (l%8) ^ (l/8)
  const int chunk = (lane % 8) ^ (lane / 8);
  const bf16_t* asrc[LA];
  const bf16_t* bsrc[LB0 + 1];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int m = min(m0 + 8 * (wave + 8 * j) + lane / 8, M - 1);
    asrc[j] = A + static_cast<size_t>(rows ? rows[m] : m) * lda + kbeg + chunk * 8;
  }
#pragma unroll
  for (int j = 0; j < LB0 + 1; ++j) {
    const int r = min(8 * (wave + 8 * j), 16 * NB - 8) + lane / 8;  // weight row of the tile
    const int n = min(cb0 * 16 + (DUAL ? r % (16 * CB) : r), N - 1);
    const bf16_t* w;
    if (DUAL) w = (r < 16 * CB ? W0 : W1) + static_cast<size_t>(n) * K;
    else w = n < N0 ? W0 + static_cast<size_t>(n) * K : W1 + static_cast<size_t>(n - N0) * K;
    bsrc[j] = w + kbeg + chunk * 8;
  }
  // The walk starts at a step that depends on the column tile and wraps around.  The
  // workgroups run nearly in step and their rows are a multiple of 4 KB apart, so unrotated every load
  // in flight has the same address bits below the row pitch (gate/up of 128 rows 47.6 -> 44.9 us, of 179 non-temporal 61.7
  // -> 56.6).  Split launches: starts that lie 8 steps apart from XCD to XCD and one apart within (one apart from tile to
  // tile, down projection of 179 rows 45.0 us; unrotated 39.8; so 38.1).  Many slices walk different ranges side by side
  // already: 64 rows in four slices are 0.2 us slower rotated, in two 0.4 us faster.  Cached weights (NT = false) gain in
  // gate/up of up to 128 rows only.
  const int rot = DUAL ? (RB <= 2 || NT ? col_tile % nkt : 0)
                       : NT && (RB >= 2 || gridDim.z <= 2) ? (col_tile % 8 * 8 + col_tile / 8) % nkt : 0;
  auto issue = [&](int stage, int kt) {
    int k = kt + rot;
    k = (k < nkt ? k : k - nkt) * 64;
#pragma unroll
    for (int j = 0; j < LA; ++j)
      __builtin_amdgcn_global_load_lds(asrc[j] + k, &lds[stage][(wave + 8 * j) * 64], 16, 0, 0);
#pragma unroll
    for (int j = 0; j < LB0; ++j)
      __builtin_amdgcn_global_load_lds(bsrc[j] + k, &lds[stage][BM * 8 + (wave + 8 * j) * 64], 16, 0, kAux);
    if (LBR > 0 && wave < LBR)
      __builtin_amdgcn_global_load_lds(bsrc[LB0] + k, &lds[stage][BM * 8 + (wave + 8 * LB0) * 64], 16, 0, kAux);
  };
  // at most `steps` steps of this wavefront's loads in flight, and its LDS reads complete
  auto wait_steps = [&](auto steps) {
    constexpr int S = decltype(steps)::value;
    if (LBR > 0 && wave < LBR) wait_vmcnt_lds<S * (LA + LB0 + 1)>();
    else wait_vmcnt_lds<S * (LA + LB0)>();
  };

  f32x4 sums[NA][RB][NB];
#pragma unroll
  for (int u = 0; u < NA; ++u)
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) sums[u][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 (&acc)[RB][NB] = sums[0];

#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nkt) issue(s, s);
  int stage = 0;
  auto step = [&](int kt, f32x4 (&sum)[RB][NB]) {
    // the loads of step kt have landed; the younger steps, at most NST - 2, stay in flight
    const int rem = nkt - 1 - kt;
    if (rem >= NST - 2) wait_steps(std::integral_constant<int, NST - 2>{});
    else if (NST > 7 && rem == 5) wait_steps(std::integral_constant<int, 5>{});
    else if (NST > 6 && rem == 4) wait_steps(std::integral_constant<int, 4>{});
    else if (NST > 5 && rem == 3) wait_steps(std::integral_constant<int, 3>{});
    else if (NST > 4 && rem == 2) wait_steps(std::integral_constant<int, 2>{});
    else if (NST > 3 && rem == 1) wait_steps(std::integral_constant<int, 1>{});
    else wait_steps(std::integral_constant<int, 0>{});
    // ... everybody's, and everybody has finished reading step kt - 1, whose stage is filled next
    __builtin_amdgcn_s_barrier();
    const int nxt = stage == 0 ? NST - 1 : stage - 1;
    if (kt + NST - 1 < nkt) issue(nxt, kt + NST - 1);
    const uint4* la = &lds[stage][0];
    const uint4* lb = &lds[stage][BM * 8];
    const int c = kk * 4 + lg;
    bf16x8 af[RB], bf[NB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int r = (wr * RB + i) * 16 + ln;
      af[i] = __builtin_bit_cast(bf16x8, la[r * 8 + (c ^ (r % 8))]);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int r = j * 16 + ln;
      bf[j] = __builtin_bit_cast(bf16x8, lb[r * 8 + (c ^ (r % 8))]);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < RB; ++i)
        sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], sum[i][j], 0, 0, 0);
    stage = stage + 1 < NST ? stage + 1 : 0;
  };
  for (int kt = 0; kt < nkt; kt += NA) {
#pragma unroll
    for (int u = 0; u < NA; ++u)
      if (u == 0 || kt + u < nkt) step(kt + u, sums[u]);
  }
#pragma unroll
  for (int u = 1; u < NA; ++u)
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] += sums[u][i][j];
  // the second halves' sums are handed over through LDS and added to the first's
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(&lds[0][0]);
  static_assert(4 * RB * NB * 64 * 16 <= NST * kStage * 16, "hand-over fits the ring");
  if (kk == 1) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) red[((wr * RB + i) * NB + j) * 64 + lane] = acc[i][j];
  }
  __syncthreads();
  if (kk == 1) return;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] += red[((wr * RB + i) * NB + j) * 64 + lane];
  float* Cs = DUAL ? nullptr : C + static_cast<size_t>(blockIdx.z) * M * N;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + (wr * RB + i) * 16 + lg * 4 + e;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        const int n = (cb0 + j) * 16 + ln;
        if (n >= N) continue;
        if (DUAL) {
          const float g = acc[i][j][e], up = acc[i][j + NB - CB][e];
          U[static_cast<size_t>(m) * N + n] = f32_to_bf16(g / (1.0f + expf(-g)) * up);
        } else {
          Cs[static_cast<size_t>(m) * N + n] = acc[i][j][e];
        }
      }
    }
}

template <int RB, int NB, int DUAL, bool FINE, bool NT>
__global__ __launch_bounds__(512) void k_gemm_ring(const bf16_t* __restrict__ A, int lda,
                                                   const int* __restrict__ rows, int M,
                                                   const bf16_t* __restrict__ W0,
                                                   const bf16_t* __restrict__ W1, int N0, int N, int K,
                                                   int k_per_slice, float* __restrict__ C,
                                                   bf16_t* __restrict__ U) {
  gemm_ring_body<RB, NB, DUAL, FINE, NT>(A, lda, rows, M, W0, W1, N0, N, K, k_per_slice, C, U);
}

// Estimated time in us of a launch of `tiles` workgroups (one per CU at a time) of 64 * rb rows x 16 * nb
// weight rows x k: the weights at the chip's stream rate, everything a CU takes in at ~40 GB/s (47 for
// 192-row tiles), or the MFMAs (rb * nb per wavefront and step, two wavefronts per SIMD).
double ring_time(long long tiles, int rb, int nb, int k) {
  const double rounds = static_cast<double>((tiles + 255) / 256);
  const double t_w = 16.0 * nb * k * 2.0 / 21.5e3;
  const double t_in = (64.0 * rb + 16.0 * nb) * k * 2.0 / (rb == 3 ? 47e3 : 40e3);
  const double t_m = k / 64.0 * 2.0 * rb * nb * 16.0 / 2400.0;
  double t = t_w > t_in ? t_w : t_in;
  if (t_m > t) t = t_m;
  return rounds * t;
}

}  // namespace

bool gemm_ring_ok(int dtype, bool operands_aligned, int lda, int K) {
  return dtype == 1 && operands_aligned && K % 64 == 0 && lda % 8 == 0;
}

// Row blocks, column blocks and slices with the lowest estimate: start + rounds of 256 workgroups (one per CU) x
// (round + step x 64-wide steps) + MB of weights / w + MB of sums / out, and what follows.  Fitted to 432 shapes (1 to 2048
// rows, 512 to 18944 columns, contraction of 896 to 18944) timed with every tile and slice count: it strays by 6 % rms; the
// tile kernels' estimates in plan_gemm are of the same form, from the same launches.
RingPlan plan_ring(int M, int N, int K, int s_cap, int force_s, bool summed) {
  struct Cost { double start, round, step, w, out; };
  static const Cost cost[3][2] = {{{2.1, 1.17, 0.244, 17.5, 3.9}, {2.3, 1.4, 0.365, 15.0, 4.8}},
                                  {{2.4, 1.3, 0.334, 18.9, 4.5}, {2.8, 1.8, 0.496, 19.8, 4.8}},
                                  {{2.75, 1.3, 0.44, 21.0, 4.5}, {3.4, 2.7, 0.66, 28.0, 5.6}}};
  const double mb_w = 2.0 * N * K / 1e6, mb_out = 4.0 * M * N / 1e6;
  RingPlan best{};
  best.t = 1e30;
  for (int rb = 1; rb <= 3; ++rb)
    for (int nb = 4; nb <= 8; nb += 4) {
      const Cost& c = cost[rb - 1][nb / 4 - 1];
      const int mt = (M + 64 * rb - 1) / (64 * rb), nt = (N + 16 * nb - 1) / (16 * nb);
      const int s_hi = force_s > 0 ? (force_s < s_cap ? force_s : s_cap) : s_cap;
      for (int S = force_s > 0 ? s_hi : 1; S <= s_hi; ++S) {
        int kps = ((K + S - 1) / S + 63) / 64 * 64;
        if (kps > K) kps = K;
        const int used = (K + kps - 1) / kps;
        const long long wg = static_cast<long long>(mt) * nt * used;
        const double t = c.start + static_cast<double>((wg + 255) / 256) * (c.round + c.step * kps / 64) + mb_w / c.w +
                         used * mb_out / c.out + slices_us(used, mb_out, summed);
        if (t < best.t * 0.98) best = RingPlan{rb, nb, used, kps, nt, mt, t};
      }
    }
  return best;
}

void launch_gemm_ring(const RingPlan& p, const bf16_t* A, int lda, const int* rows, int M, const bf16_t* W0,
                      const bf16_t* W1, int N0, int N, int K, float* C, bool fine, bool once, hipStream_t st) {
  const dim3 grid(p.nt, p.mt, p.S);
  const bool nt = once && p.mt == 1;
#define DLLMC_RL(RB, NB, FINE, NT)                                                                                  \
  hipLaunchKernelGGL((k_gemm_ring<RB, NB, 0, FINE, NT>), grid, dim3(512), 0, st, A, lda, rows, M, W0, W1, N0, N, K, \
                     p.kps, C, nullptr)
#define DLLMC_R(RB, NB)                     \
  do {                                      \
    if (fine) DLLMC_RL(RB, NB, true, false); \
    else if (nt) DLLMC_RL(RB, NB, false, true); \
    else DLLMC_RL(RB, NB, false, false);    \
  } while (0)
  switch (p.rb * 10 + p.nb) {
    case 14: DLLMC_R(1, 4); break;
    case 18: DLLMC_R(1, 8); break;
    case 24: DLLMC_R(2, 4); break;
    case 28: DLLMC_R(2, 8); break;
    case 34: DLLMC_R(3, 4); break;
    default: DLLMC_R(3, 8); break;
  }
#undef DLLMC_R
#undef DLLMC_RL
}

// Columns per workgroup: whole rounds over the CUs.  48 for an FFN width of 12288 (256 workgroups), 80 for
// 18944 (237: 51 us, 48 columns in two rounds 61), 16 for 3072.
void plan_ring_swiglu(int M, int m, int K, int& rb, int& cb) {
  rb = cb = 1;
  double best_t = 1e30;
  for (int r = 1; r <= 3; ++r)
    for (int c = 1; c <= 5; ++c) {
      const long long tiles = static_cast<long long>((M + 64 * r - 1) / (64 * r)) * ((m + 16 * c - 1) / (16 * c));
      const double t = ring_time(tiles, r, 2 * c, K);
      if (t < best_t * 0.98) { best_t = t; rb = r; cb = c; }
    }
}

void launch_gemm_ring_swiglu(const bf16_t* A, int lda, const int* rows, int M, const bf16_t* w_gate,
                             const bf16_t* w_up, int m, int K, bf16_t* u, bool once, hipStream_t st) {
  int rb, cb;
  plan_ring_swiglu(M, m, K, rb, cb);
  const dim3 grid((m + 16 * cb - 1) / (16 * cb), (M + 64 * rb - 1) / (64 * rb), 1);
#define DLLMC_R(RB, CB)                                                                                      \
  do {                                                                                                       \
    if (once && grid.y == 1)                                                                                 \
      hipLaunchKernelGGL((k_gemm_ring<RB, 2 * CB, 1, false, true>), grid, dim3(512), 0, st, A, lda, rows, M, w_gate, \
                         w_up, m, m, K, K, nullptr, u);                                                      \
    else                                                                                                     \
      hipLaunchKernelGGL((k_gemm_ring<RB, 2 * CB, 1, false, false>), grid, dim3(512), 0, st, A, lda, rows, M, w_gate, \
                         w_up, m, m, K, K, nullptr, u);                                                      \
  } while (0)
#define DLLMC_RC(RB)                 \
  switch (cb) {                      \
    case 1: DLLMC_R(RB, 1); break;   \
    case 2: DLLMC_R(RB, 2); break;   \
    case 3: DLLMC_R(RB, 3); break;   \
    case 4: DLLMC_R(RB, 4); break;   \
    default: DLLMC_R(RB, 5); break;  \
  }
  if (rb == 1) { DLLMC_RC(1) }
  else if (rb == 2) { DLLMC_RC(2) }
  else { DLLMC_RC(3) }
#undef DLLMC_RC
#undef DLLMC_R
}

}  // namespace dllmc
