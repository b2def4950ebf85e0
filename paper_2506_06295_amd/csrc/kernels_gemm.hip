// Gathered linear maps  C[i, :] = A[rows[i], :] * W^T  (W row-major [N, K], K contiguous).
//
// Kernels:
//  * k_gemm_simple  -- plain LDS-tiled FMA kernel for any storage type and shape: the fallback
//                      for shapes and alignments that the MFMA kernels do not take (float32
//                      models: kernels_gemm_f32.hip).
//  * k_gemm_ring    -- bf16 MFMA kernel for few activation rows against a weight matrix that is read
//                      exactly once from HBM, and for any column count: kernels_gemm_ring.hip.
//  * k_gemm_wide / k_gemm_mid -- bf16 MFMA kernels for launches with hundreds of activation rows whose operands both go
//                      through LDS by direct global->LDS loads: tiles of 128 x 128 to 256 x 256 in one workgroup per
//                      CU (gemm_wide.hpp), also with SwiGLU, V-verify and Q | K epilogues, and 128 x 128 tiles in two per CU, also
//                      with V-verify's epilogue and the head's reduction (k_gemm_mid_vverify, k_gemm_mid_head).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.hpp"

namespace dllmc {


int gemm_max_slices() { return kMaxSlices; }

// ------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_gemm_simple(const T* __restrict__ A, int lda,
                                                     const int* __restrict__ rows, int M,
                                                     const T* __restrict__ W0,
                                                     const T* __restrict__ W1, int N0, int N, int K,
                                                     float* __restrict__ C) {
  __shared__ float As[16][65];
  __shared__ float Ws[16][65];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int e = threadIdx.x; e < 1024; e += 256) {
      const int r = e / 16, kk = e % 16;
      float a = 0.f, w = 0.f;
      if (k0 + kk < K) {
        const int m = m0 + r;
        if (m < M) {
          const int row = rows ? rows[m] : m;
          a = ldf(A + static_cast<size_t>(row) * lda + k0 + kk);
        }
        const int nn = n0 + r;
        if (nn < N) {
          const T* wp = nn < N0 ? W0 + static_cast<size_t>(nn) * K
                                : W1 + static_cast<size_t>(nn - N0) * K;
          w = ldf(wp + k0 + kk);
        }
      }
      As[kk][r] = a;
      Ws[kk][r] = w;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Ws[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int nn = n0 + tx * 4 + j;
      if (nn < N) C[static_cast<size_t>(m) * N + nn] = acc[i][j];
    }
  }
}

// ------------------------------------------------------------------------------------
// LDS-direct MFMA kernels for many activation rows (refresh steps, the V projection of all
// response rows, batched sequences), where the work is bound by the matrix cores and by L2
// rather than by the weight stream.  Workgroup = WM x WN wavefronts, each (16*MI) rows x
// (16*NJ) columns of v_mfma_f32_16x16x32_bf16 accumulators.  Both operands reach LDS with
// global_load_lds_dwordx4 (no VGPR staging): a wavefront instruction copies 8 rows x 128
// contiguous bytes (64 values of the contraction index) into 1 KB of LDS in lane order, i.e.
// LDS holds [row][8 slots of 16 bytes]; the slot of chunk c of row r is c ^ (r % 8) so that
// the 16-byte fragment reads of 8 consecutive rows hit 8 different bank groups.  Two LDS
// stages (128-row tiles) or a ring of slots per operand (192- and 256-row tiles, gemm_wide_body): later steps'
// loads are in flight while step t is multiplied.
// Rows beyond M read a valid row again and are dropped at the store.
//   fat: 2 x 2 wavefronts of 128 x 128 -> 256 x 256 tile (every byte pulled from L2 feeds 128
//        flops), all 160 KB of LDS, one workgroup per CU: M >= fat_min_m.
//   mid: 2 x 2 wavefronts of  64 x 64 -> 128 x 128 tile, 64 KB of LDS, two workgroups per CU:
//        enough tiles to fill the chip when M is a few hundred rows.
constexpr int kFatM = 256, kFatN = 256, kFatK = 64;
constexpr int kMidM = 128, kMidN = 128;

//   PAIR = 1 (gemm_wide_body; fused gate/up + SwiGLU, single slice): the tile's weight rows are BN/2 rows of W0
//        (gate) followed by the same BN/2 rows of W1 (up), so every lane ends up with the gate
//        and the up sum of the same output element and stores bf16(silu(gate) * up) to U[M, N]
//        (N = FFN width; the grid has N / (BN/2) column tiles).
//   EPI = 1 / 2 (single slice): the step's work on the tile is finished in the epilogue, nothing
//        goes through float32 slices and no row kernel follows.
//        1: V-verify (Sec. 3.2.2, Eq. cos_sim).  Activation row i is carried row i of the step
//           (position first + i % per_seq of sequence i / per_seq); the sums are rounded to bf16,
//           scored against the cached row they replace (per row and 64-column block the three
//           sums go to `part`, laid out as for k_vverify_tile) and written to the cache.
//        2: (gemm_wide_body) Q | K with RoPE.  A tile column block of 128 is one head, two column wavefronts; the
//           weight rows are dealt so that a lane's accumulators j and j + 2 hold the rotation pair
//           (t, t + 64): rotated in registers, query heads go to the compact q_out[i] and the
//           other heads to cache row rows[i].
//        3: vocabulary projection of the head: the tile's logits are reduced per row
//           (head_tile_reduce), to the entries at C.
struct TileEpilogue {
  // EPI = 1
  int first, per_seq, n, L_p;
  bf16_t* cache;         // V cache [*, N] (EPI 1); K (or V) cache [*, d_kv] (EPI 2)
  float* part;           // tile sums, or nullptr: no scoring
  int part_stride, metric;
  const int* rmap;       // paged layout: cache row of a logical row, or nullptr
  // EPI = 2
  const float2* tab;     // [n][64] (cos, sin)
  bf16_t* q_out;         // [M, N0]
  int d_kv, rope_second;
};

}  // namespace dllmc
#include "gemm_wide.hpp"
namespace dllmc {

// Head: a tile of logits in LDS (128 columns per row, column c of row r at c ^ 16 * (r / 4 % 4): the four
// rows that a wavefront stores at once hit different banks) is reduced per row to (maximum, sum of
// exp, first index of the maximum) by TPR neighbouring threads and stored to part[row * tiles + tile].
// The results cross through LDS for this: reducing them in the accumulator layout, 16 lanes to a row,
// takes four times the vector instructions.
// The exponentials are the hardware's 2^x of a float32 product: 6e-8 |l - maximum| relative on a term that weighs
// exp(l - maximum), so at most ~3e-7 of the sum, less than adding 64 terms in float32 costs.  Confidences against 64 bits, rms
// (expf in its place): 100 rows of 126464 9.78e-6 (9.78e-6), 128 of 152064 1.88e-6 (1.87e-6), 100 of 4096 6.8e-7 (7.0e-7);
// 190.5 us (195.5) for the first.
template <int TPR>
__device__ __forceinline__ void head_tile_reduce(const float* tile, int m0, int M, int col_tile, int tiles,
                                                 HeadPart* __restrict__ part) {
  constexpr int CPT = 128 / TPR;  // columns per thread
  constexpr float kLog2e = 1.4426950408889634f;
  const int r = threadIdx.x / TPR, c0 = (threadIdx.x % TPR) * CPT;
  const int swz = ((r >> 2) & 3) << 4;
  float v[CPT];
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < CPT / 4; ++t) {
    // (neighbouring rows start at different pieces of their columns: other banks)
    const int c = c0 + 4 * ((t + r) % (CPT / 4));
    const float4 f = *reinterpret_cast<const float4*>(&tile[r * 128 + (c ^ swz)]);
    v[4 * t] = f.x; v[4 * t + 1] = f.y; v[4 * t + 2] = f.z; v[4 * t + 3] = f.w;
    mx = fmaxf(mx, fmaxf(fmaxf(f.x, f.y), fmaxf(f.z, f.w)));
  }
  const float mu = mx == -INFINITY ? 0.f : mx;
  float sum = 0.f;
  int first = 0x7fffffff;
#pragma unroll
  for (int t = 0; t < CPT / 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sum += __builtin_amdgcn_exp2f((v[4 * t + e] - mu) * kLog2e);
      if (v[4 * t + e] == mx) first = min(first, c0 + 4 * ((t + r) % (CPT / 4)) + e);
    }
  if (first == 0x7fffffff) first = c0;  // nothing but NaN
#pragma unroll
  for (int o = 1; o < TPR; o <<= 1) {
    const float om = __shfl_xor(mx, o, 64), os = __shfl_xor(sum, o, 64);
    const int oa = __shfl_xor(first, o, 64);
    const float nm = fmaxf(mx, om), nu = nm == -INFINITY ? 0.f : nm;
    const float fs = mx == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mx - nu) * kLog2e);
    const float fo = om == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((om - nu) * kLog2e);
    first = mx > om ? first : (om > mx ? oa : min(first, oa));
    sum = sum * fs + os * fo;
    mx = nm;
  }
  if (threadIdx.x % TPR == 0 && m0 + r < M)
    part[static_cast<size_t>(m0 + r) * tiles + col_tile] = HeadPart{mx, sum, col_tile * 128 + first, 0};
}

template <int WM, int WN, int MI, int NJ, int EPI = 0, bool FINE = false, bool NT = false>
__device__ __forceinline__ void gemm_lds_body(const bf16_t* __restrict__ A, int lda,
                                              const int* __restrict__ rows, int M,
                                              const bf16_t* __restrict__ W0,
                                              const bf16_t* __restrict__ W1, int N0, int N, int K,
                                              int k_per_slice, float* __restrict__ C,
                                              const TileEpilogue* ep = nullptr, int starts = 8) {
  constexpr int NWV = WM * WN;
  constexpr int BM = WM * MI * 16, BN = WN * NJ * 16;
  constexpr int LA = BM / 8 / NWV, LB = BN / 8 / NWV;  // load instructions per wavefront and step
  static_assert(BM % (8 * NWV) == 0 && BN % (8 * NWV) == 0, "loader must divide evenly");
  // NT: non-temporal weight loads, where a single row tile reads weights that no cache will hold at their next use (see
  // k_gemm_ring; with two row tiles to a weight tile they cost the second one its hits: head of 200 rows 294 -> 354 us)
  constexpr int kAux = NT ? 2 : 0;
  // [stage][activation rows, then weight rows][8 slots], 16 bytes each
  // (EPI: followed by two ints per tile row, see below.  One LDS object on purpose: with a second
  // one the compiler can no longer tell the fragment reads from the loads in flight into the
  // other stage and waits for those before every read.)
  constexpr int kStage = (BM + BN) * 8;
  // Two workgroups per CU (128 x 128, four wavefronts), two stages of both operands: the loads of step kt+1 go out before
  // the wait for step kt and a second barrier at the end of the step protects the stage they overwrite (a five-slot loop
  // with 16 KB slots measured 3-8 % slower).
  constexpr int kLdsTotal = 2 * kStage + (EPI == 1 ? 2 * BM / 4 : 0);
  __shared__ __attribute__((aligned(1024))) uint4 lds_all[kLdsTotal];
  uint4 (*lds)[kStage] = reinterpret_cast<uint4 (*)[kStage]>(lds_all);
  int (*meta)[BM] = reinterpret_cast<int (*)[BM]>(lds_all + 2 * kStage);
  // (the wavefront index as a scalar: the LDS addresses of the loads, which go through M0, are then
  // scalar arithmetic instead of vector instructions and v_readfirstlane in every step)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  const int wm = wave / WN, wn = wave % WN;
  int col_tile, row_tile;
  xcd_tile_map_blocked(col_tile, row_tile);
  const int m0 = row_tile * BM, n0 = col_tile * BN;
  const int kbeg = blockIdx.z * k_per_slice;
  const int klen = min(K, kbeg + k_per_slice) - kbeg;  // multiple of kFatK
  const int nkt = klen / kFatK;

  // loader: instruction q of an operand covers rows [8q, 8q+8); wavefront w issues
  // q = L*w .. L*w+L-1.  Lane l: row 8q + l/8, LDS slot l%8, global chunk (l%8) ^ (row%8).
  const bf16_t* asrc[LA];
  const bf16_t* bsrc[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int r = 8 * (LA * wave + j) + lane / 8;
    const int chunk = (lane % 8) ^ (r % 8);
    int m = m0 + r;
    if (m >= M) m = M - 1;
    int row;
    if (EPI == 1) row = (m / ep->per_seq) * ep->n + ep->first + m % ep->per_seq;
    else row = rows ? rows[m] : m;
    asrc[j] = A + static_cast<size_t>(row) * lda + kbeg + chunk * 8;
  }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int r = 8 * (LB * wave + j) + lane / 8;
    const int chunk = (lane % 8) ^ (r % 8);
    const int nn = n0 + r;  // < N: N % BN == 0
    bsrc[j] = (nn < N0 ? W0 + static_cast<size_t>(nn) * K
                       : W1 + static_cast<size_t>(nn - N0) * K) + kbeg + chunk * 8;
  }
  // EPI 1: what the epilogue needs to know about the tile's rows -- cache row, index of the row's score (-1: not
  // scored) -- looked up here so that the trips to memory pass under the main loop.
  if (EPI == 1 && threadIdx.x < BM) {
    const int r = threadIdx.x;
    const int m = min(m0 + r, M - 1);
    const int seq = m / ep->per_seq, pos = ep->first + m % ep->per_seq;
    const int row = seq * ep->n + pos;
    meta[0][r] = ep->rmap ? ep->rmap[row] : row;
    meta[1][r] = (m0 + r < M && ep->part != nullptr && pos >= ep->L_p)
                     ? seq * (ep->n - ep->L_p) + (pos - ep->L_p) : -1;
  }
#define DLLMC_LDS_ISSUE(stage, kt)                                                              \
  {                                                                                             \
    _Pragma("unroll") for (int j = 0; j < LA; ++j) __builtin_amdgcn_global_load_lds(            \
        asrc[j] + (kt) * kFatK, &lds[stage][(LA * wave + j) * 64], 16, 0, 0);                   \
    _Pragma("unroll") for (int j = 0; j < LB; ++j) __builtin_amdgcn_global_load_lds(            \
        bsrc[j] + (kt) * kFatK, &lds[stage][BM * 8 + (LB * wave + j) * 64], 16, 0, kAux);       \
  }

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The walk over the contraction index starts at a step that depends on the XCD and wraps
  // around: the workgroups of a launch run nearly in step and their rows are a multiple of 4 KB
  // apart, so unrotated every load in flight on the chip has the same address bits below the row
  // pitch and the memory channels are loaded unevenly (4096 x 4096 x 16384: 959 -> 1097 TFLOP/s).
  // The workgroups of one XCD keep a common start, they share operand blocks through its L2.
  // starts: 8, or 1 where every tile has to begin at the same step -- equal rows of the vocabulary projection have to give
  // equal logits whatever tile they are in, so that the lowest token wins, and a sum's bits depend on where its walk begins
  const int rot = (((blockIdx.x + gridDim.x * blockIdx.y) & (starts - 1)) * nkt) >> 3;
  DLLMC_LDS_ISSUE(0, rot)
  // (FINE, see k_gemm_ring: the first and the second half of the steps in sums of their own.  Halves, because even and odd
  // steps apart, two copies of the loop body in turn, took a third longer.)
  auto step = [&](int kt, f32x4 (&sum)[MI][NJ]) {
    const int cur = kt & 1;
    const bool more = kt + 1 < nkt;
    {
      if (more) {
        DLLMC_LDS_ISSUE(cur ^ 1, kt + 1 + rot < nkt ? kt + 1 + rot : kt + 1 + rot - nkt)
        wait_vmcnt<LA + LB>();  // this wavefront's loads of step kt have landed
      } else {
        wait_vmcnt<0>();
      }
      // bare barrier (no memory fence: a fence would wait for the loads of step kt+1 as well)
      __builtin_amdgcn_s_barrier();  // ... and everybody else's
    }
    const uint4* la = &lds[cur][0];
    const uint4* lb = &lds[cur][BM * 8];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int c = kk * 4 + lg;  // 16-byte chunk of the 64-wide step this lane group multiplies
      bf16x8 af[MI], bf[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = wm * (MI * 16) + i * 16 + ln;
        af[i] = __builtin_bit_cast(bf16x8, la[r * 8 + (c ^ (r % 8))]);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int r = wn * (NJ * 16) + j * 16 + ln;
        bf[j] = __builtin_bit_cast(bf16x8, lb[r * 8 + (c ^ (r % 8))]);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], sum[i][j], 0, 0, 0);
    }
    // all fragment reads of this stage are complete before the loads issued at the top of the
    // next iteration overwrite it.  The explicit wait matters: without it the compiler puts the
    // wait for the last reads (and the MFMAs they feed) behind the barrier, and a load that hits
    // in L1 (the neighbouring workgroup on the CU reads the same activation rows) can land
    // before those reads execute.
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  if (FINE) {
    f32x4 late[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) late[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int half = nkt / 2;
    int kt = 0;
    for (; kt < half; ++kt) step(kt, acc);
    for (; kt < nkt; ++kt) step(kt, late);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] += late[i][j];
  } else {
    for (int kt = 0; kt < nkt; ++kt) step(kt, acc);
  }
#undef DLLMC_LDS_ISSUE

  if (EPI == 3) {
    static_assert(EPI != 3 || (BN == 128 && BM * 128 * sizeof(float) <= sizeof(lds_all)), "the tile fits");
    __syncthreads();  // everybody has finished the fragment reads of the last step
    float* tile = reinterpret_cast<float*>(lds_all);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tile[(wm * (MI * 16) + i * 16 + lg * 4 + e) * 128 + ((wn * (NJ * 16) + j * 16 + ln) ^ (lg << 4))] =
              acc[i][j][e];
    __syncthreads();
    head_tile_reduce<NWV * 64 / BM>(tile, m0, M, col_tile, gridDim.x, reinterpret_cast<HeadPart*>(C));
    return;
  }
  if (EPI == 1) {
    // V-verify, finished on the tile.  A wavefront's 16-row x 64-column block of
    // results (rounded to bf16) is staged through a private piece of LDS so that it leaves, and
    // the cached rows it is compared with arrive, as 16-byte pieces of contiguous row segments:
    // lane l then holds columns 8*(l%8) .. +8 of block rows l/8 and l/8 + 8.
    static_assert(EPI != 1 || NJ == 4, "a wavefront's block is 64 columns wide");
    constexpr int kStg = 72;  // staging row stride in elements: 64 columns + 16 bytes
    static_assert(NWV * 16 * kStg * sizeof(bf16_t) <= kStage * sizeof(uint4), "staging fits a stage");
    __syncthreads();  // everybody has finished the fragment reads of the last step
    uint32_t* stg32 = reinterpret_cast<uint32_t*>(&lds[0][0]) + wave * (16 * kStg / 2);
    const bf16_t* stg = reinterpret_cast<const bf16_t*>(stg32);
    const int rr = lane / 8, ch = lane % 8;
    const int odd = ln & 1;
    const int n_ct = N / 64, ct = col_tile * WN + wn;
    uint4 old[2];  // the old rows of block i, requested one block ahead
    auto request = [&](int i) {
      const int rb = wm * (MI * 16) + i * 16;  // first row of the block inside the tile
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          old[h] = make_uint4(0u, 0u, 0u, 0u);
          const int r = rb + rr + 8 * h;
          if (meta[1][r] >= 0)
            old[h] = *reinterpret_cast<const uint4*>(ep->cache + static_cast<size_t>(meta[0][r]) * N + n0 +
                                                     wn * 64 + ch * 8);
        }
    };
    request(0);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int rb = wm * (MI * 16) + i * 16;
      // final values of the lane's accumulator elements
      float val[NJ][4];
      uint4 old_i[2] = {old[0], old[1]};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) val[j][e] = acc[i][j][e];
      if (i + 1 < MI) request(i + 1);
      // Neighbouring lanes hold neighbouring columns of the same four rows: they trade one value
      // of each row pair, after which the even lane owns columns (ln, ln + 1) of row e and the odd
      // lane columns (ln - 1, ln) of row e + 1, one 32-bit store each.
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float got = dpp_xor1(odd ? val[j][e] : val[j][e + 1]);
          const float lo = odd ? got : val[j][e];
          const float hi = odd ? val[j][e + 1] : got;
          const int r = lg * 4 + e + odd;
          stg32[(r * kStg + j * 16 + (ln & ~1)) / 2] = pack_bf16x2(lo, hi);
        }
      // the wavefront's own stores have completed before its loads are issued
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = rb + rr + 8 * h;  // row inside the tile
        const uint4 nv = *reinterpret_cast<const uint4*>(stg + (rr + 8 * h) * kStg + ch * 8);
        const int crow = meta[0][r];
        {
          const int sidx = meta[1][r];
          if (ep->part != nullptr) {  // uniform
            const uint32_t nw4[4] = {nv.x, nv.y, nv.z, nv.w};
            const uint32_t ow4[4] = {old_i[h].x, old_i[h].y, old_i[h].z, old_i[h].w};
            float dot = 0.f, nn = 0.f, no = 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const float a0 = __uint_as_float(nw4[t] << 16), a1 = __uint_as_float(nw4[t] & 0xffff0000u);
              const float b0 = __uint_as_float(ow4[t] << 16), b1 = __uint_as_float(ow4[t] & 0xffff0000u);
              if (ep->metric == 0) {
                dot += a0 * b0; nn += a0 * a0; no += b0 * b0;
                dot += a1 * b1; nn += a1 * a1; no += b1 * b1;
              } else {
                const float d0 = a0 - b0, d1 = a1 - b1;
                dot += d0 * d0;
                dot += d1 * d1;
              }
            }
            // the eight lanes of a row: pairs, quads, then the two quads
            dot += dpp_xor1(dot); nn += dpp_xor1(nn); no += dpp_xor1(no);
            dot += dpp_xor2(dot); nn += dpp_xor2(nn); no += dpp_xor2(no);
            dot += dpp_half_mirror(dot); nn += dpp_half_mirror(nn); no += dpp_half_mirror(no);
            if (sidx >= 0 && ch == 0) {
              ep->part[(static_cast<size_t>(0) * n_ct + ct) * ep->part_stride + sidx] = dot;
              ep->part[(static_cast<size_t>(1) * n_ct + ct) * ep->part_stride + sidx] = nn;
              ep->part[(static_cast<size_t>(2) * n_ct + ct) * ep->part_stride + sidx] = no;
            }
          }
          if (m0 + r < M)
            *reinterpret_cast<uint4*>(ep->cache + static_cast<size_t>(crow) * N + n0 + wn * 64 + ch * 8) = nv;
        }
      }
      // ... and the loads before the next block's stores
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return;
  }
  float* Cs = C + static_cast<size_t>(blockIdx.z) * M * N;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + wm * (MI * 16) + i * 16 + lg * 4 + e;
      if (m < M) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          Cs[static_cast<size_t>(m) * N + n0 + wn * (NJ * 16) + j * 16 + ln] = acc[i][j][e];
      }
    }
}

// The tile kernels of one workgroup per CU (gemm_wide_body): 2 x 2 wavefronts of 16 MI x 16 NJ, tiles of 32 MI x 32 NJ.
template <int MI, int NJ>
__global__ __launch_bounds__(256) void k_gemm_wide(const bf16_t* __restrict__ A, int lda, const int* __restrict__ rows, int M,
                                                   const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int N0, int N,
                                                   int K, int k_per_slice, float* __restrict__ C, int starts) {
  gemm_wide_body<2, 2, MI, NJ>(A, lda, rows, M, W0, W1, N0, N, K, k_per_slice, C, nullptr, nullptr, starts);
}
// gate/up + SwiGLU: N is the FFN width, a tile has 16 NJ columns of each
template <int MI, int NJ>
__global__ __launch_bounds__(256) void k_gemm_wide_swiglu(const bf16_t* __restrict__ A, int lda, const int* __restrict__ rows,
                                                          int M, const bf16_t* __restrict__ Wg, const bf16_t* __restrict__ Wu,
                                                          int N, int K, bf16_t* __restrict__ U) {
  gemm_wide_body<2, 2, MI, NJ, 1>(A, lda, rows, M, Wg, Wu, N, N, K, K, nullptr, U);
}
// tile kernels that finish the step's work in their epilogue (single slice): V-verify and Q | K with RoPE (see EPI above)
template <int WM, int WN, int MI, int NJ>
__global__ __launch_bounds__(256) void k_gemm_wide_vverify(const bf16_t* __restrict__ A, int lda, int M,
                                                           const bf16_t* __restrict__ W, int N, int K, TileEpilogue ep) {
  gemm_wide_body<WM, WN, MI, NJ, 0, 1>(A, lda, nullptr, M, W, nullptr, N, N, K, K, nullptr, nullptr, &ep);
}
template <int MI, int NJ>
__global__ __launch_bounds__(256) void k_gemm_wide_qk(const bf16_t* __restrict__ A, int lda, const int* __restrict__ rows, int M,
                                                      const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int N0,
                                                      int N, int K, TileEpilogue ep) {
  gemm_wide_body<2, 2, MI, NJ, 0, 2>(A, lda, rows, M, W0, W1, N0, N, K, K, nullptr, nullptr, &ep);
}

__global__ __launch_bounds__(256) void k_gemm_mid(const bf16_t* __restrict__ A, int lda,
                                                  const int* __restrict__ rows, int M,
                                                  const bf16_t* __restrict__ W0,
                                                  const bf16_t* __restrict__ W1, int N0, int N,
                                                  int K, int k_per_slice, float* __restrict__ C, int starts) {
  gemm_lds_body<2, 2, 4, 4>(A, lda, rows, M, W0, W1, N0, N, K, k_per_slice, C, nullptr, starts);
}

__global__ __launch_bounds__(256) void k_gemm_mid_fine(const bf16_t* __restrict__ A, int lda,
                                                       const int* __restrict__ rows, int M,
                                                       const bf16_t* __restrict__ W0,
                                                       const bf16_t* __restrict__ W1, int N0, int N,
                                                       int K, int k_per_slice, float* __restrict__ C) {
  gemm_lds_body<2, 2, 4, 4, 0, true>(A, lda, rows, M, W0, W1, N0, N, K, k_per_slice, C);
}

__global__ __launch_bounds__(256) void k_gemm_mid_vverify(const bf16_t* __restrict__ A, int lda, int M,
                                                          const bf16_t* __restrict__ W, int N, int K,
                                                          TileEpilogue ep) {
  gemm_lds_body<2, 2, 4, 4, 1>(A, lda, nullptr, M, W, nullptr, N, N, K, K, nullptr, &ep);
}

template <bool NT>
__global__ __launch_bounds__(256) void k_gemm_mid_head(const bf16_t* __restrict__ A, int lda, int M,
                                                       const bf16_t* __restrict__ W, int N, int K,
                                                       float* __restrict__ C) {
  gemm_lds_body<2, 2, 4, 4, 3, false, NT>(A, lda, nullptr, M, W, nullptr, N, N, K, K, C, nullptr, 1);
}

// 256 rows x (48 gate + 48 up) columns, four wavefronts of 64 x 96 each: for up to 256 rows and
// an FFN width that is a multiple of 48 the grid is one workgroup per 48 columns (12288 / 48 =
// 256, one per CU), where the 128 x 128 tiles leave half of the CUs with twice the work (a
// response refresh of 256 rows: 80 -> 69 us per layer; two workgroups of 128 x 96 per CU: 73; with non-temporal
// weight loads 65.7 -> 62.7; with the body of one wavefront per SIMD 55).
template <bool NT>
__global__ __launch_bounds__(256) void k_gemm_tall_swiglu(const bf16_t* __restrict__ A, int lda,
                                                          const int* __restrict__ rows, int M,
                                                          const bf16_t* __restrict__ Wg,
                                                          const bf16_t* __restrict__ Wu, int N, int K,
                                                          bf16_t* __restrict__ U) {
  gemm_wide_body<4, 1, 4, 6, 1, 0, NT>(A, lda, rows, M, Wg, Wu, N, N, K, K, nullptr, U);
}

// V floats per thread; every slice's load is issued before the first addition (a loop over the runtime count waits
// for each), slices in order.
template <int V, int S>
__global__ __launch_bounds__(256) void k_reduce_slices(const float* __restrict__ c_part, size_t MN,
                                                       float* __restrict__ out) {
  const size_t i = (static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x) * V;
  if (i >= MN) return;
  if (V == 4) {
    f32x4 u[S];
#pragma unroll
    for (int s = 0; s < S; ++s) u[s] = *reinterpret_cast<const f32x4*>(c_part + static_cast<size_t>(s) * MN + i);
#pragma unroll
    for (int s = 1; s < S; ++s) u[0] += u[s];
    *reinterpret_cast<f32x4*>(out + i) = u[0];
  } else {
    float u[S];
#pragma unroll
    for (int s = 0; s < S; ++s) u[s] = c_part[static_cast<size_t>(s) * MN + i];
#pragma unroll
    for (int s = 1; s < S; ++s) u[0] += u[s];
    out[i] = u[0];
  }
}

void launch_reduce_slices(const float* c_part, int S, int M, int N, float* out, hipStream_t st) {
  const size_t MN = static_cast<size_t>(M) * N;
  if (MN == 0) return;
  const bool vec = MN % 4 == 0 &&
                   ((reinterpret_cast<uintptr_t>(c_part) | reinterpret_cast<uintptr_t>(out)) & 15u) == 0;
  const dim3 grid(static_cast<unsigned>((MN + (vec ? 1023 : 255)) / (vec ? 1024 : 256)));
#define DLLMC_RS(Sv)                                                                                         \
  case Sv:                                                                                                   \
    if (vec) hipLaunchKernelGGL((k_reduce_slices<4, Sv>), grid, dim3(256), 0, st, c_part, MN, out);           \
    else hipLaunchKernelGGL((k_reduce_slices<1, Sv>), grid, dim3(256), 0, st, c_part, MN, out);               \
    break;
  switch (S) {
    DLLMC_RS(1) DLLMC_RS(2) DLLMC_RS(3) DLLMC_RS(4) DLLMC_RS(5) DLLMC_RS(6) DLLMC_RS(7) DLLMC_RS(8)
    default: break;  // no more than kMaxSlices
  }
#undef DLLMC_RS
}

// ------------------------------------------------------------------------------------
namespace {
// The process default (guarded by a mutex: contexts copy it at creation, dllmc_set_gemm_tuning
// writes it) and the settings in force on this thread: a context's own copy while one of its
// calls runs (TuningScope), else a snapshot of the default taken by the calling launcher.
GemmTuning g_default_tune;
std::mutex g_tune_mu;
thread_local const GemmTuning* t_scope = nullptr;
thread_local GemmTuning t_snapshot;
const GemmTuning& tune() {
  if (t_scope) return *t_scope;
  std::lock_guard<std::mutex> lock(g_tune_mu);
  t_snapshot = g_default_tune;
  return t_snapshot;
}
#define g_tune (tune())

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
}  // namespace

static thread_local bool t_last_stream = false;
bool gemm_last_was_stream() { return t_last_stream; }
void gemm_clear_last_stream() { t_last_stream = false; }

#undef g_tune
GemmTuning gemm_default_tuning() {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  return g_default_tune;
}
TuningScope::TuningScope(const GemmTuning* t) : prev(t_scope) { t_scope = t; }
TuningScope::~TuningScope() { t_scope = prev; }

void gemm_set_tile_min_m(int m) { std::lock_guard<std::mutex> lock(g_tune_mu); if (m > 0) g_default_tune.tile_min_m = m; }
void gemm_set_fat_min_m(int m) { std::lock_guard<std::mutex> lock(g_tune_mu); if (m > 0) g_default_tune.fat_min_m = m; }

void gemm_set_tuning(int force_s, int target_wg) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  if (force_s >= 0) g_default_tune.force_s = force_s;
  if (target_wg > 0) g_default_tune.target_wg = target_wg;
}
#define g_tune (tune())

// Shapes of k_gemm_wide and their estimates: us = start + rounds over the 256 CUs x (round + step x 64-wide steps) + MB of
// weights / kWideW + MB of float32 results / out.  Fitted to 6048 launches (200 to 12288 rows, maps of 896 x 2432 to 3584 x 18944 and
// 4096 x 12288, one to eight slices, cold weights; 6 to 7 % rms).
struct WideShape { int bm, bn; double start, round, step, out; };
constexpr double kWideW = 23;
constexpr WideShape kWide[6] = {{256, 256, 1.37, 3.46, 1.179, 6.8}, {192, 256, 1.88, 2.4, 0.931, 6.8},
                                {256, 128, 2.53, 0.72, 0.712, 4.8}, {128, 256, 2.94, 0.3, 0.757, 5.3},
                                {192, 128, 2.46, 0.3, 0.605, 4.6}, {128, 128, 2.13, 0.3, 0.478, 4.6}};

// Which kernel, how many slices of the contraction index and how long a slice: pure host logic.
struct GemmPlan {
  int kind;  // 0 nothing fits, 1 plain, 2 weight-streaming, 3 LDS-direct tiles of one workgroup per CU, 4 128x128
             // LDS-direct of two, 7 float32 on the matrix cores
  int wide;  // kind 3: index into kWide
  int S, kps, nt, mt;
  double t;       // estimated us (kinds 2, 3 and 4)
  RingPlan ring;  // kind 2
  F32Plan f32;    // kind 7
};

GemmPlan plan_gemm(int dtype, bool operands_aligned, int lda, int M, int N, int N0, int K,
                   size_t c_capacity, bool summed) {
  GemmPlan p{};
  const size_t MN = static_cast<size_t>(M) * N;
  if (M <= 0 || N <= 0 || K <= 0 || c_capacity < MN) return p;
  // most slices the caller's buffer can hold
  const int s_cap = static_cast<int>(c_capacity / MN < static_cast<size_t>(kMaxSlices)
                                         ? c_capacity / MN : static_cast<size_t>(kMaxSlices));
  if (dtype == 0 && operands_aligned && K % 4 == 0 && lda % 4 == 0) {
    p.kind = 7;
    p.f32 = plan_f32(M, N, K, s_cap, g_tune.force_s);
    p.S = p.f32.S; p.kps = p.f32.kps; p.nt = p.f32.nt; p.mt = p.f32.mt;
    return p;
  }
  if (!gemm_ring_ok(dtype, operands_aligned, lda, K)) {
    p.kind = 1; p.S = 1; p.kps = K; p.nt = (N + 63) / 64; p.mt = (M + 63) / 64;
    return p;
  }
  const GemmTuning defaults;
  const bool fat_ok = M >= g_tune.fat_min_m && N % kFatN == 0 && N0 % kFatN == 0;
  const bool mid_ok = M >= g_tune.tile_min_m && N % kMidN == 0 && N0 % kMidN == 0;  // (and the other shapes of k_gemm_wide)
  if (fat_ok || mid_ok) {
    // The estimate of plan_ring for the tile kernels (kWide; 128 x 128 with two workgroups per CU: a round of up to 256 has each
    // CU to itself), at every slice count.  In a step (198 maps of 200 to 12288 rows, with what reads the sums) the choice among
    // them is 0.6 % from the quickest (with prices fitted to tiles whose last blocks came twice and whose sums left in rows of 16
    // bytes 3.5 %).  op_linear: a price for the launch that adds slices, in place of a plain rule on rows alone: 192 rows x 4096 x 4096 20.6 us, so 18.2;
    // 333 x 3072 x 1024 19.2 -> 9.9; 400 x 2432 x 896 15.2 -> 9.5; 1536 x 896 x 2432 25.2 -> 17.8; 64 x 12288 x 4096 31.7 -> 26.1.  Over 208
    // shapes (16 to 2048 rows, eleven maps) it takes 0.7 % less with kWide's present prices than with those, nowhere more than 1.5 % more.
    const bool literal = g_tune.force_s > 0 || g_tune.fat_min_m != defaults.fat_min_m ||
                         g_tune.tile_min_m != defaults.tile_min_m || g_tune.target_wg != defaults.target_wg;
    double best = 1e30;
    auto offer = [&](int kind, int wide, int S) {
      const int bm = wide < 0 ? kMidM : kWide[wide].bm, bn = wide < 0 ? kMidN : kWide[wide].bn;
      int kps = ((K + S - 1) / S + kFatK - 1) / kFatK * kFatK;
      if (kps > K) kps = K;
      const int used = (K + kps - 1) / kps, mt = (M + bm - 1) / bm, nt = N / bn;
      const long long wg = static_cast<long long>(mt) * nt * used;
      const double steps = kps / kFatK, mb_w = 2.0 * N * K / 1e6, mb_out = 4.0 * M * N / 1e6, rem = wg % 512;
      double t = kind == 3 ? kWide[wide].start + static_cast<double>((wg + 255) / 256) * (kWide[wide].round + kWide[wide].step * steps) +
                                 mb_w / kWideW + used * mb_out / kWide[wide].out
                           : 3.05 + (wg / 512 * 0.89 + (rem == 0 ? 0.0 : rem <= 256 ? 0.58 : 0.89)) * steps + mb_w / 20 +
                                 used * mb_out / 6.3;
      t += slices_us(used, mb_out, summed);
      if (t < best * 0.98) {
        best = t;
        p.kind = kind; p.wide = wide; p.S = used; p.kps = kps; p.nt = nt; p.mt = mt; p.t = t;
      }
    };
    const bool only_fat = literal && fat_ok;  // thresholds and slice counts set by the caller
    const int s_lo = g_tune.force_s > 0 ? (g_tune.force_s < s_cap ? g_tune.force_s : s_cap) : 1;
    int s_hi = g_tune.force_s > 0 ? s_lo : s_cap, m_lo = s_lo, m_hi = s_hi;
    if (g_tune.force_s <= 0 && g_tune.target_wg != defaults.target_wg) {
      const int tiles = ((M + kMidM - 1) / kMidM) * (N / kMidN);
      m_lo = m_hi = std::max(1, std::min(s_cap, g_tune.target_wg / tiles));
    }
    for (int S = s_lo; fat_ok && S <= s_hi; ++S)
      if (S == s_lo || K / S >= 8 * kFatK) offer(3, 0, S);
    for (int S = m_lo; mid_ok && !only_fat && S <= m_hi; ++S)
      if (S == m_lo || K / S >= 8 * kFatK) offer(4, -1, S);
    // (not for sums that are the caller's result: the 128 x 128 kernel deals them to two per element)
    for (int i = 1; i < 6 && !summed && !literal; ++i)
      for (int S = s_lo; N % kWide[i].bn == 0 && N0 % 8 == 0 && S <= s_hi; ++S)
        if (S == s_lo || K / S >= 8 * kFatK) offer(3, i, S);
    if (!literal) {
      const RingPlan r = plan_ring(M, N, K, s_cap, 0, summed);
      // (168 maps of 192 to 1024 rows, cold, with what reads their sums: the choice is 0.7 % from the quicker of both on average)
      if (r.t < best * (summed ? 0.98 : 1.0)) {
        p.kind = 2; p.ring = r; p.S = r.S; p.kps = r.kps; p.nt = r.nt; p.mt = r.mt; p.t = r.t;
      }
    }
    return p;
  }
  p.kind = 2;
  p.ring = plan_ring(M, N, K, s_cap, g_tune.force_s, summed);
  p.S = p.ring.S; p.kps = p.ring.kps; p.nt = p.ring.nt; p.mt = p.ring.mt; p.t = p.ring.t;
  return p;
}

int gemm_plan_slices(int dtype, int M, int N, int N0, int K, size_t c_capacity) {
  return plan_gemm(dtype, true, K, M, N, N0, K, c_capacity, false).S;
}

int launch_gemm(int dtype, const void* A, int lda, const int* rows, int M, const void* W0,
                const void* W1, int N0, int N, int K, float* c_part, size_t c_capacity,
                hipStream_t st, bool summed, float* whole, bool logits) {
  t_last_stream = false;
  if (M <= 0 || N <= 0) return 1;
  const bool al = aligned16(A) && aligned16(W0) && (W1 == nullptr || aligned16(W1));
  const GemmPlan p = plan_gemm(dtype, al, lda, M, N, N0, K, c_capacity, summed);
  if (p.kind == 0 || static_cast<size_t>(p.S) * M * N > c_capacity) return 0;  // nothing launched
  t_last_stream = p.kind == 2;
  if (whole != nullptr && p.S == 1) c_part = whole;
  const bf16_t* a = static_cast<const bf16_t*>(A);
  const bf16_t* w0 = static_cast<const bf16_t*>(W0);
  const bf16_t* w1 = static_cast<const bf16_t*>(W1);
  const dim3 grid(p.nt, p.mt, p.S);
  const int starts = logits ? 1 : 8;
  switch (p.kind) {
    case 1:
      if (dtype == 1)
        hipLaunchKernelGGL(k_gemm_simple<bf16_t>, grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, N0,
                           N, K, c_part);
      else
        hipLaunchKernelGGL(k_gemm_simple<float>, grid, dim3(256), 0, st,
                           static_cast<const float*>(A), lda, rows, M,
                           static_cast<const float*>(W0), static_cast<const float*>(W1), N0, N, K,
                           c_part);
      break;
    case 2:
      launch_gemm_ring(p.ring, a, lda, rows, M, w0, w1, N0, N, K, c_part, summed, g_tune.weights_once && !logits, st);
      break;
    case 7:
      launch_gemm_f32(p.f32, static_cast<const float*>(A), lda, rows, M, static_cast<const float*>(W0),
                      static_cast<const float*>(W1), N0, N, K, c_part, st);
      break;
    case 3:
#define DLLMC_W(MI, NJ) \
  hipLaunchKernelGGL((k_gemm_wide<MI, NJ>), grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, N0, N, K, p.kps, c_part, starts)
      switch (p.wide) {
        case 0: DLLMC_W(8, 8); break;
        case 1: DLLMC_W(6, 8); break;
        case 2: DLLMC_W(8, 4); break;
        case 3: DLLMC_W(4, 8); break;
        case 4: DLLMC_W(6, 4); break;
        default: DLLMC_W(4, 4); break;
      }
#undef DLLMC_W
      break;
    case 4:
      if (summed)
        hipLaunchKernelGGL(k_gemm_mid_fine, grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, N0, N, K, p.kps, c_part);
      else
        hipLaunchKernelGGL(k_gemm_mid, grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, N0, N, K, p.kps, c_part, starts);
      break;
  }
  return p.S;
}

int launch_gemm_head(int dtype, const void* A, int lda, int M, const void* W, int N, int K, HeadPart* part,
                     size_t part_capacity, hipStream_t st) {
  // The 128 x 128 tile kernel whatever the number of rows: with a single row it streams the weights at 5.9
  // TB/s (op_head of 1 / 64 / 100 / 128 rows x 126464 x 4096: 184 / 190 / 196 / 203 us; the streaming kernel
  // with the same reduction 213 / 227 / 247 / 250), two workgroups per CU and loads of whole lines.
  // From 641 rows the 256 x 256 tiles are ahead in spite of the logits' trip through memory (513 rows 645
  // against 690 us, 700 rows 779 against 750).
  if (dtype != 1 || K % kFatK || N % kMidN || lda % 8 || M > 640) return 0;
  if (!aligned16(A) || !aligned16(W) || !aligned16(part)) return 0;
  if (static_cast<size_t>(M) * (N / kMidN) > part_capacity) return 0;
  t_last_stream = false;
  // (weights beyond the memory-side cache: 100 rows x 126464 x 4096 191 -> 180 us, 4 rows 178 -> 163)
  const bool nt = M <= kMidM && static_cast<size_t>(N) * K * 2 > kMemorySideCache;
  hipLaunchKernelGGL(nt ? k_gemm_mid_head<true> : k_gemm_mid_head<false>, dim3(N / kMidN, (M + kMidM - 1) / kMidM),
                     dim3(256), 0, st, static_cast<const bf16_t*>(A), lda, M, static_cast<const bf16_t*>(W), N, K,
                     reinterpret_cast<float*>(part));
  return N / kMidN;
}

// Gate/up of many rows: the LDS-direct tile kernels with paired gate/up column blocks, one slice; the tile shape with the lowest
// estimate, of the form of kWide's (rows and columns of each matrix).  The weights' term (w) differs between shapes by more than any
// rate could: it is what the fit leaves to it, and none of it counts for the choice (one price for all, 0.40 % from the
// quickest shape; this table 0.38).  Over 872 launches of 200 to 12288 rows and FFN widths 1536 to 18944 it is 5 to 7 % rms
// and 0.4 % from the quickest shape on average, 8 at worst.
struct PairTile { int rows, cols; double start, round, step, w, out; };
constexpr PairTile kPairTiles[10] = {
    {256, 128, 1.9, 3.27, 1.349, 318, 2.1}, {256, 96, 0.5, 3.3, 1.038, 30, 2.3}, {192, 96, 1.1, 2.0, 0.866, 20, 2.0},
    {192, 128, 2.7, 0.65, 1.045, 35, 1.6}, {256, 64, 1.5, 1.54, 0.761, 30, 1.6}, {128, 128, 1.2, 2.16, 0.797, 37, 2.1},
    {192, 64, 1.9, 1.13, 0.654, 54, 1.8}, {128, 96, 0.6, 2.0, 0.614, 13, 1.9}, {128, 64, 1.1, 0.88, 0.503, 25, 1.8},
    {256, 48, 1.9, 1.3, 0.72, 50, 2.0}};
int swiglu_shape(int M, int m, int K) {
  int pick = -1;
  double best = 1e30;
  for (int i = 0; i < 10; ++i) {
    const PairTile& p = kPairTiles[i];
    if (m % p.cols || (i == 0 && M < g_tune.fat_min_m) || (i == 9 && M > 256)) continue;
    const long long n = static_cast<long long>((M + p.rows - 1) / p.rows) * (m / p.cols);
    const double t = p.start + static_cast<double>((n + 255) / 256) * (p.round + p.step * (K / kFatK)) +
                     4e-6 * m * K / p.w + 2e-6 * M * m / p.out;
    if (t < best) { best = t; pick = i; }
  }
  return pick;
}

bool launch_gemm_swiglu(int dtype, const void* A, int lda, const int* rows, int M,
                        const void* w_gate, const void* w_up, int m, int K, void* u,
                        hipStream_t st) {
  if (M <= 0 || m <= 0) return true;
  if (dtype == 0) {
    if (!gemm_f32_ok(A, lda, w_gate, w_up, K)) return false;
    t_last_stream = false;
    return launch_gemm_f32_swiglu(static_cast<const float*>(A), lda, rows, M,
                                  static_cast<const float*>(w_gate), static_cast<const float*>(w_up), m, K,
                                  static_cast<float*>(u), st);
  }
  if (!gemm_ring_ok(dtype, aligned16(A) && aligned16(w_gate) && aligned16(w_up), lda, K)) return false;
  if (M >= g_tune.tile_min_m) {
    const int pick = swiglu_shape(M, m, K);
    if (pick >= 0) {
      t_last_stream = false;
      const bf16_t* a = static_cast<const bf16_t*>(A);
      const bf16_t* w0 = static_cast<const bf16_t*>(w_gate);
      const bf16_t* w1 = static_cast<const bf16_t*>(w_up);
      bf16_t* uo = static_cast<bf16_t*>(u);
      const dim3 grid(m / kPairTiles[pick].cols, (M + kPairTiles[pick].rows - 1) / kPairTiles[pick].rows, 1);
#define DLLMC_SW(...) hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, m, K, uo)
      switch (pick) {
        case 0: DLLMC_SW(k_gemm_wide_swiglu<8, 8>); break;
        case 1: DLLMC_SW(k_gemm_wide_swiglu<8, 6>); break;
        case 2: DLLMC_SW(k_gemm_wide_swiglu<6, 6>); break;
        case 3: DLLMC_SW(k_gemm_wide_swiglu<6, 8>); break;
        case 4: DLLMC_SW(k_gemm_wide_swiglu<8, 4>); break;
        case 5: DLLMC_SW(k_gemm_wide_swiglu<4, 8>); break;
        case 6: DLLMC_SW(k_gemm_wide_swiglu<6, 4>); break;
        case 7: DLLMC_SW(k_gemm_wide_swiglu<4, 6>); break;
        case 8: DLLMC_SW(k_gemm_wide_swiglu<4, 4>); break;
        default:  // one row tile
          if (g_tune.weights_once) DLLMC_SW(k_gemm_tall_swiglu<true>);
          else DLLMC_SW(k_gemm_tall_swiglu<false>);
          break;
      }
#undef DLLMC_SW
      return true;
    }
  }
  t_last_stream = true;
  launch_gemm_ring_swiglu(static_cast<const bf16_t*>(A), lda, rows, M, static_cast<const bf16_t*>(w_gate),
                          static_cast<const bf16_t*>(w_up), m, K, static_cast<bf16_t*>(u),
                          g_tune.weights_once, st);
  return true;
}

// The way through V-verify that takes least, by estimates in us with what follows the launch (launch_scores_from_part, or the row
// kernel; in a step the selection adds the sums, which spares the former's launch).  One launch: start + rounds over the 256
// CUs x (round + step x 64-wide steps) + MB of weights / w + MB of V / out.  489 shapes (32 to 12288 rows, 64 to 8192 columns,
// contraction of 512 to 8192, cold weights) were timed each way: rms 13 % (64 x 64; priced low where it and the split are
// level, 200 and 256 rows x 4096 x 4096 22.5 and 24.7 us against 23.8 and 23.4), 3 (128 x 128 with two workgroups per CU), 6 (192 x 64), 4 (the
// others), 8 (split).  The single operation takes 0.8 % longer than the quickest way on average, 5 % or more in 19 shapes; with prices fitted to
// tiles of eight wavefronts and V-verify's epilogue as a surcharge on kWide's it was 2.5 % (4608 rows x 2048 x 2048 58.7
// us, so 46.2; 3300 x 2560 x 2560 73.2, 57.8; 12288 x 1024 x 1024 42.5, 34.6).
VPlan plan_vverify(int dtype, bool operands_aligned, int lda, int M, int N, int K, size_t c_capacity, bool in_step) {
  VPlan best{kVSplit, 0, 0, 0.0};
  if (dtype != 1 || M < 1 || !operands_aligned || lda % 8 || K % kFatK || N % 64) return best;
  struct Tile { int way, bm, bn; double start, round, step, w, out; };
  constexpr Tile tiles[6] = {{kVFused, 64, 64, 4.7, 2.2, 0.184, 23, 1.24}, {kVMid, kMidM, kMidN, 7.5, 2.15, 0.817, 12, 2.92},
                             {kVMid, 128, 256, 4.8, 6.59, 0.672, 9.6, 2.91}, {kVR192, 192, 64, 4.9, 1.9, 0.412, 8.6, 1.83},
                             {kVR192, 192, 256, 3.9, 8.43, 0.988, 14, 4.79}, {kVFat, 256, 256, 4.7, 13.86, 1.157, 11, 4.64}};
  const double steps = K / kFatK, mb_w = 2.0 * N * K / 1e6, mb_v = 2.0 * M * N / 1e6;
  best.us = 1e30;
  for (const Tile& t : tiles) {
    if (N % t.bn || (t.bm > 64 && M < g_tune.tile_min_m) || (t.way == kVFat && M < g_tune.fat_min_m)) continue;
    const long long n = static_cast<long long>((M + t.bm - 1) / t.bm) * (N / t.bn);
    double rounds = static_cast<double>((n + 255) / 256), walks = rounds;
    if (t.bm == kMidM && t.bn == kMidN) {  // two workgroups per CU; up to 256 in the last round have each CU to themselves
      rounds = static_cast<double>((n + 511) / 512);
      walks = rounds - (n % 512 != 0 && n % 512 <= 256 ? 0.31 : 0.0);
    }
    const double us = t.start + rounds * t.round + walks * t.step * steps + mb_w / t.w + mb_v / t.out;
    if (us < best.us) best = VPlan{t.way, t.bm, t.bn, us};
  }
  const GemmPlan p = plan_gemm(dtype, true, lda, M, N, N, K, c_capacity, false);
  const double split = 3.7 + p.t + mb_v / 7.3 + M / 300.0;
  // (against 64 x 64 tiles of 192 to 511 rows the split has to be 6 % ahead: its price is that much low there, 192 rows x 2048 x 2048
  // 14.6 us, the tiles 13.4; 333 x 128 x 896 9.4 and 8.6)
  const double bar = best.us * (best.way == kVFused && M >= g_tune.tile_min_m && M < g_tune.fat_min_m ? 0.94 : 1.0);
  if (p.kind != 0 && split < bar - (in_step ? 2.0 : 0.0)) best = VPlan{kVSplit, 0, 0, split};
  return best;
}

// Shape of kWide whose tiles finish Q | K of M rows x N columns in one slice, -1: none (every shape that divides the
// columns would leave more than a quarter of the CUs without a workgroup).  By the estimates of the plain maps, with 4 us per
// round and the bf16 results at 5 MB / us for the epilogue: 7 % rms over 756 launches (200 to 12288 rows, seven widths), the choice 0.04 %
// from the quickest shape on average (at worst 1.6).
int qk_tile_shape(int M, int N, int N0, int K) {
  if (K % kFatK || M < g_tune.tile_min_m) return -1;
  const int cus = 256, least = 3 * cus / 4;
  int shape = -1;
  double best = 1e30;
  for (int i = 0; i < 6; ++i) {
    const WideShape& w = kWide[i];
    if (N % w.bn || N0 % 128 || (i == 0 && M < g_tune.fat_min_m)) continue;
    const long long tiles = static_cast<long long>((M + w.bm - 1) / w.bm) * (N / w.bn);
    if (tiles < least) continue;
    const double t = w.start + static_cast<double>((tiles + cus - 1) / cus) * (w.round + 4.0 + w.step * (K / kFatK)) +
                     2e-6 * N * K / kWideW + 2e-6 * M * N / 5.0;
    if (t < best) { best = t; shape = i; }
  }
  return shape;
}

void launch_gemm_vverify_tiles(const VPlan& plan, const void* A, int lda, int M, int first, int per_seq, int n,
                               int L_p, const void* W, int N, int K, void* v_cache, float* part,
                               int part_stride, int metric, const int* rmap, hipStream_t st) {
  TileEpilogue ep{};
  ep.first = first; ep.per_seq = per_seq; ep.n = n; ep.L_p = L_p;
  ep.cache = static_cast<bf16_t*>(v_cache);
  ep.part = part; ep.part_stride = part_stride; ep.metric = metric; ep.rmap = rmap;
  t_last_stream = false;
  const bf16_t* a = static_cast<const bf16_t*>(A);
  const bf16_t* w = static_cast<const bf16_t*>(W);
  const dim3 grid(N / plan.bn, (M + plan.bm - 1) / plan.bm);
#define DLLMC_V(...) hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(256), 0, st, a, lda, M, w, N, K, ep)
  switch (plan.bm * 1000 + plan.bn) {
    case 256256: DLLMC_V(k_gemm_wide_vverify<2, 2, 8, 8>); break;
    case 192256: DLLMC_V(k_gemm_wide_vverify<2, 2, 6, 8>); break;
    case 128256: DLLMC_V(k_gemm_wide_vverify<2, 2, 4, 8>); break;
    case 192064: DLLMC_V(k_gemm_wide_vverify<4, 1, 3, 4>); break;
    default: DLLMC_V(k_gemm_mid_vverify); break;
  }
#undef DLLMC_V
}

bool launch_gemm_qk_tiles(int dtype, const void* A, int lda, const int* rows, int M, const void* wq,
                          const void* w2, int d_q, int d_kv, int d_h, int K, const float2* rope_tab,
                          int n, void* q_out, void* cache, bool rope_second, const int* rmap,
                          hipStream_t st) {
  if (M <= 0) return true;
  if (dtype != 1 || d_h != 128 || lda % 8 || !aligned16(A) || !aligned16(wq) || !aligned16(w2)) return false;
  const int N = d_q + d_kv;
  const int shape = qk_tile_shape(M, N, d_q, K);
  if (shape < 0) return false;
  TileEpilogue ep{};
  ep.n = n; ep.cache = static_cast<bf16_t*>(cache); ep.rmap = rmap; ep.tab = rope_tab;
  ep.q_out = static_cast<bf16_t*>(q_out); ep.d_kv = d_kv; ep.rope_second = rope_second ? 1 : 0;
  t_last_stream = false;
  const bf16_t* a = static_cast<const bf16_t*>(A);
  const bf16_t* w0 = static_cast<const bf16_t*>(wq);
  const bf16_t* w1 = static_cast<const bf16_t*>(w2);
  const dim3 grid(N / kWide[shape].bn, (M + kWide[shape].bm - 1) / kWide[shape].bm, 1);
#define DLLMC_QK(MI, NJ) hipLaunchKernelGGL((k_gemm_wide_qk<MI, NJ>), grid, dim3(256), 0, st, a, lda, rows, M, w0, w1, d_q, N, K, ep)
  switch (shape) {
    case 0: DLLMC_QK(8, 8); break;
    case 1: DLLMC_QK(6, 8); break;
    case 2: DLLMC_QK(8, 4); break;
    case 3: DLLMC_QK(4, 8); break;
    case 4: DLLMC_QK(6, 4); break;
    default: DLLMC_QK(4, 4); break;
  }
#undef DLLMC_QK
  return true;
}

int plan_tile(int launch, int M, int N, int N0, int K, int* cols) {
  int rows = 0, c = 0;
  if (launch == 1) {
    const int i = M >= g_tune.tile_min_m && gemm_ring_ok(1, true, K, K) ? swiglu_shape(M, N, K) : -1;
    if (i >= 0) { rows = kPairTiles[i].rows; c = kPairTiles[i].cols; }
  } else if (launch == 2) {
    const int i = qk_tile_shape(M, N, N0, K);
    if (i >= 0) { rows = kWide[i].bm; c = kWide[i].bn; }
  } else {
    const size_t slices = static_cast<size_t>(M) * N * kMaxSlices;
    const GemmPlan p = plan_gemm(1, true, K, M, N, N0, K, slices, false);
    if (launch == 0 && p.kind == 3) { rows = kWide[p.wide].bm; c = kWide[p.wide].bn; }
    if (launch == 3) {
      const VPlan v = plan_vverify(1, true, K, M, N, K, slices, true);
      if (v.way != kVFused && !(v.bm == kMidM && v.bn == kMidN)) { rows = v.bm; c = v.bn; }
    }
  }
  if (cols) *cols = c;
  return rows;
}

#undef g_tune

}  // namespace dllmc
