// Body of the LDS-direct tile kernels with one workgroup per CU (tiles of 128, 192 and 256 rows), included by kernels_gemm.hip.
//
// Four wavefronts, one per SIMD, of 16 MI rows x 16 NJ columns each.  Operands, LDS layout and the meaning of PAIR, EPI and
// NT are those of gemm_lds_body; where results are bf16 the products are taken as W A^T, so that a lane holds four neighbouring
// columns of one row and every result leaves as 8- or 16-byte pieces.  Float32 sums are taken as A W^T: of 16-byte pieces in rows of
// their own no two share a request, and a 256 x 256 tile took 5.4 us to store (a launch of 64 tiles, one step: 15.4 us, so 12.0).
//
// Bound by the matrix cores and the power they may draw: a 256 x 256 x 64 step of nothing but MFMAs takes 0.89 us on zeros and
// 1.03 on random data (8 wavefronts; 32 x 32 x 16 MFMAs 1.10), with the fragment reads, the barrier and loads that
// always hit 1.01 and 1.14.  This loop: 0.96 and 1.35 (4096 x 4096 x 4096 .. 12288, slope); eight wavefronts of 128 x 64 with
// the reads of 16 MFMAs ahead 1.11 and 1.46, as two groups that multiply and load in turn the same.  What counts:
//   * 128 x 128 per wavefront reads 128 KB of fragments per step from LDS, 128 x 64 192 KB;
//   * with one wavefront per SIMD nothing else fills the matrix pipe, so the reads of the next 32 contraction values and the
//     loads go out singly between MFMAs (2.5 MFMAs apart; in groups of four reads and four loads 1.43 and 1.69, loads every second
//     MFMA 1.01 and 1.37).  The last steps, which have nothing to load, are copies of the loop's body; while they loaded
//     the last block again a launch was 1 to 3 us longer;
//   * what the V-verify and Q | K epilogues look up comes in one trip in front of the first loads (with a branch for the row
//     list and the row map around each it was up to sixteen, one after the other), what they compare or rotate with under the
//     last MFMAs, and results leave 16 bytes at a time.  Q | K (us; with trips one by one, so, with eight wavefronts): 8192 rows x 8192 x 4096
//     452, 434, 430; 8192 x 4096 x 2048 138, 120, 118; 8192 x 2048 x 1024 49, 41, 40.  V-verify: 12288 x 4096 x 4096 344, 336, 340;
//     4608 x 4096 x 4096 165, 157, 175; 4096 x 4096 x 512 44, 40, 39.6;
//   * gate/up's epilogue, see silu_mul.  In the step (us, eight wavefronts / so): gate/up of 4608 rows x 12288 x 4096 735 / 694, of
//     1024 185 / 160, of 768 156 / 133, of 256 64 / 55; down projection of 1024 rows 92 / 81;
//   * the accumulators are held in the accumulation registers by the constraint of an asm statement: left to the
//     compiler, which has 256 of them and 130 other live registers, 48 to 540 moves enter the loop (none now; a move inside
//     the loop would have to keep 8 wait states from the asm statement whose result it reads).
#pragma once

namespace dllmc {
namespace {

// silu(g) * up, bit for bit what g / (1 + expf(-g)) * up gives (32 million gates of either sign, 1e-41 to 110: none differs; at
// most 2.1 units in the last place), in 45 ns per value and wavefront instead of 54: the quotient by a reciprocal and one
// residual.  A quarter, because the reciprocal of more than 2^126 (gates below -87.3) would be flushed to zero; the
// fix-up for infinities.  (With an exponential of 2^t and no range reduction 37 ns, but 4 units, and nothing left below -87.3.)
__device__ __forceinline__ float silu_mul(float g, float up) {
  const float d = 1.f + expf(-g);
  const float c = 0.25f * __builtin_amdgcn_rcpf(0.25f * d);
  const float q = g * c;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, d, g), c, q), d, g) * up;
}

// Depths of the rings of BM and BN rows (128 bytes each): 1280 rows in all.
template <int BM, int BN> struct WideRing {
  static constexpr int kWhole = 1280 / (BM + BN);  // of both
  static constexpr int kLeft = 1280 - kWhole * (BM + BN);
  static constexpr int DA = kWhole + (kLeft >= BM && (BM >= BN || kLeft < BN) ? 1 : 0);
  static constexpr int DB = kWhole + (DA == kWhole && kLeft >= BN ? 1 : 0);
};

template <int WM, int WN, int MI, int NJ, int PAIR = 0, int EPI = 0, bool NT = false>
__device__ __forceinline__ void gemm_wide_body(const bf16_t* __restrict__ A, int lda, const int* __restrict__ rows, int M,
                                               const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int N0, int N,
                                               int K, int k_per_slice, float* __restrict__ C, bf16_t* __restrict__ U = nullptr,
                                               const TileEpilogue* ep = nullptr, int starts = 8) {
  constexpr int BM = WM * MI * 16, BN = WN * NJ * 16;
  constexpr int LA = BM / 32, LB = BN / 32;  // load instructions per wavefront and step
  static_assert(WM * WN == 4 && BM % 32 == 0 && BN % 32 == 0, "four wavefronts, whole load instructions");
  static_assert(!PAIR || NJ % 2 == 0, "gate and up column blocks come in pairs");
  static_assert(EPI == 0 || (NJ % 4 == 0 && (EPI == 1 || WN * NJ % 8 == 0)), "blocks of 64 columns; a head is two");
  constexpr int kAux = NT ? 2 : 0;
  constexpr bool kPlain = EPI == 0 && !PAIR;
  // A ring of LDS slots for each operand's blocks of 64 contraction values, as deep as 160 KB allow.  The barrier of step
  // kt -- everybody has read all of A(kt) and B(kt), everybody's loads of step kt + 1 have landed -- stands between the two
  // halves of the step and makes room for the next block of operand X, loaded during the second half, and of operand
  // Y, the one with the deeper ring, loaded during the first half of the next step.  256 x 256: X = B two deep, Y = A three;
  // A(kt+2) stays in flight across the barrier.
  typedef WideRing<BM, BN> Ring;
  constexpr int DA = Ring::DA, DB = Ring::DB;
  constexpr bool XB = DA >= DB;  // X is B
  constexpr int DX = XB ? DB : DA, DY = XB ? DA : DB, LX = XB ? LB : LA, LY = XB ? LA : LB;
  constexpr int kSlotA = BM * 8, kSlotB = BN * 8;
  static_assert((DA * kSlotA + DB * kSlotB) * sizeof(uint4) <= 160 * 1024 && DX >= 2 && DX <= 5, "LDS of one CU");
  __shared__ __attribute__((aligned(1024))) uint4 lds[DA * kSlotA + DB * kSlotB];  // A's slots, then B's
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  const int wm = wave / WN, wn = wave % WN;
  int col_tile, row_tile;
  xcd_tile_map_blocked(col_tile, row_tile);
  const int m0 = row_tile * BM, n0 = col_tile * (PAIR ? BN / 2 : BN);
  const int kbeg = blockIdx.z * k_per_slice;
  const int nkt = (min(K, kbeg + k_per_slice) - kbeg) / kFatK;

  // loader: wavefront w issues instructions L*w .. L*w+L-1 of an operand, 8 rows each; lane l: row l/8, slot l%8, global
  // chunk (l%8) ^ (row%8)
  const bf16_t* asrc[LA];
  const char* bbase[LB];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int r = 8 * (LA * wave + j) + lane / 8;
    const int m = min(m0 + r, M - 1);
    int row;
    if (EPI == 1) row = (m / ep->per_seq) * ep->n + ep->first + m % ep->per_seq;
    else row = rows ? rows[m] : m;
    asrc[j] = A + static_cast<size_t>(row) * lda + kbeg + ((lane % 8) ^ (r % 8)) * 8;
  }
  // The 8 weight rows of an instruction are consecutive rows of one matrix (the tile origins and the W0 | W1 boundary
  // are multiples of 8): the address is a scalar base plus the same lane offset for every instruction.
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int r = 8 * (LB * wave + j);
    const bf16_t* w;
    if (PAIR) {
      w = (r < BN / 2 ? W0 : W1) + static_cast<size_t>(n0 + r % (BN / 2)) * K;
    } else {
      // EPI 2: LDS weight row 64 b + 16 j + c is column (j/2)*64 + (b%2)*32 + (j%2)*16 + c of head b/2 of the tile, so
      // that a lane's accumulators j and j + 2 are rotation pairs
      const int nn = n0 + (EPI == 2 ? (r / 128) * 128 + ((r % 64) / 32) * 64 + ((r / 64) % 2) * 32 + r % 32 : r);
      w = nn < N0 ? W0 + static_cast<size_t>(nn) * K : W1 + static_cast<size_t>(nn - N0) * K;
    }
    bbase[j] = wave_uniform_ptr(reinterpret_cast<const char*>(w + kbeg));
  }
  const uint32_t boff = static_cast<uint32_t>((lane / 8) * K + ((lane % 8) ^ (lane / 8)) * 8) * sizeof(bf16_t);
  // the walk starts at a step that depends on the XCD, see gemm_lds_body
  const int rot = (((blockIdx.x + gridDim.x * blockIdx.y) & (starts - 1)) * nkt) >> 3;
  auto kof = [&](int kt) { const int k = kt + rot; return (k < nkt ? k : k - nkt) * kFatK; };
  auto issue_a = [&](int slot, int ko, int j) {
    __builtin_amdgcn_global_load_lds(asrc[j] + ko, &lds[slot * kSlotA + (LA * wave + j) * 64], 16, 0, 0);
  };
  // (the scalar sum re-read as a wavefront constant and the offset through an empty asm: otherwise the compiler folds the
  // two into per-lane pointers)
  auto issue_b = [&](int slot, int ko, int j) {
    const char* bp = wave_uniform_ptr(bbase[j] + ko * static_cast<int>(sizeof(bf16_t)));
    uint32_t o = boff;
    asm volatile("" : "+v"(o));
    __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(bp + o),
                                     &lds[DA * kSlotA + slot * kSlotB + (LB * wave + j) * 64], 16, 0, kAux);
  };
  auto issue_x = [&](int slot, int ko, int j) { if (XB) issue_b(slot, ko, j); else issue_a(slot, ko, j); };
  auto issue_y = [&](int slot, int ko, int j) { if (XB) issue_a(slot, ko, j); else issue_b(slot, ko, j); };
  auto block_x = [&](int t) {
    const int ko = kof(t);
    if (t >= nkt) return;
#pragma unroll
    for (int j = 0; j < LX; ++j) issue_x(t, ko, j);
  };
  auto block_y = [&](int t) {
    const int ko = kof(t);
    if (t >= nkt) return;
#pragma unroll
    for (int j = 0; j < LY; ++j) issue_y(t, ko, j);
  };
  // row of this lane's elements of block i; their columns are 16 j + 4 lg .. + 3 of the wavefront's
  auto row_of = [&](int i) { return m0 + wm * (MI * 16) + i * 16 + ln; };
  // EPI: cache row of every block's row, and its position (EPI 2), looked up in front of the first blocks -- a register that is
  // waited for behind them waits for all of them -- and all at once
  int crow[MI], meta[MI];
  if (EPI != 0) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int m = min(row_of(i), M - 1);
      crow[i] = EPI == 1 ? (m / ep->per_seq) * ep->n + ep->first + m % ep->per_seq : m;
    }
    if (EPI == 2 && rows != nullptr) {
#pragma unroll
      for (int i = 0; i < MI; ++i) crow[i] = rows[crow[i]];
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
      if (EPI == 2) meta[i] = crow[i] % ep->n;
    if (ep->rmap != nullptr) {
#pragma unroll
      for (int i = 0; i < MI; ++i) crow[i] = ep->rmap[crow[i]];
    }
    if (EPI == 1) {  // rows that are not scored: the complement
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int m = row_of(i);
        if (m >= M || ep->part == nullptr || ep->first + m % ep->per_seq < ep->L_p) crow[i] = ~crow[i];
      }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      asm volatile("" : "+v"(crow[i]));
      if (EPI == 2) asm volatile("" : "+v"(meta[i]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // in the order of the main loop: X(t), Y(t + DY - DX); Y(DY - 1) goes out in step 0
#pragma unroll
  for (int t = 0; t < DY - DX; ++t) block_y(t);
#pragma unroll
  for (int t = 0; t < DX - 1; ++t) {
    block_x(t);
    block_y(t + DY - DX);
  }
  block_x(DX - 1);
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  bf16x8 af[2][MI], bf[2][NJ];
  // q-th fragment of 32 contraction values: the weights' and the first activations' are needed first
  auto read = [&](int slot_a, int slot_b, int kk, int q) {
    const int c = kk * 4 + lg;
    if (q < NJ) {
      const int r = PAIR ? (q / (NJ / 2)) * (BN / 2) + wn * (NJ / 2 * 16) + (q % (NJ / 2)) * 16 + ln : wn * (NJ * 16) + q * 16 + ln;
      bf[kk][q] = __builtin_bit_cast(bf16x8, lds[DA * kSlotA + slot_b * kSlotB + r * 8 + (c ^ (r % 8))]);
    } else {
      const int r = wm * (MI * 16) + (q - NJ) * 16 + ln;
      af[kk][q - NJ] = __builtin_bit_cast(bf16x8, lds[slot_a * kSlotA + r * 8 + (c ^ (r % 8))]);
    }
  };
  // The MFMAs of 32 contraction values; `between` gets the number of those before it.  The compiler does not know how long the
  // results of an asm statement take (8 wait states: it puts s_nop 7 between the builtin and a store of its result) and may read
  // accumulators as soon as the loop ends: the last statement of a step waits itself.  Inside the loop nothing but these statements
  // may touch them (no moves; with the last four MFMAs left to the compiler it moved their results right in front of a statement that
  // reads them).
  auto half = [&](auto kk_, auto&& between) {
    constexpr int kk = decltype(kk_)::value;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bf16x8 &x = kPlain ? af[kk][i] : bf[kk][j], &y = kPlain ? bf[kk][j] : af[kk][i];
        if (kk == 1 && i * NJ + j == MI * NJ - 1)
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 7" : "+a"(acc[i][j]) : "v"(x), "v"(y));
        else
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(x), "v"(y));
        __builtin_amdgcn_sched_barrier(0);
        between(i * NJ + j);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  // reads and loads are spread over this many MFMAs, so that the last have time to land (256 x 256: three quarters of them
  // 1 to 2 % slower; the others up to 4 % faster)
  constexpr int kSpan = MI * NJ >= 64 ? MI * NJ * 5 / 8 : MI * NJ * 3 / 4;

  // X(0) and Y(0) have landed
  if (nkt >= DY) wait_vmcnt_lds<(DX - 1) * LX + (DY > DX ? DX - 1 : DX - 2) * LY>();
  else wait_vmcnt_lds<0>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int q = 0; q < MI + NJ; ++q) read(0, 0, 0, q);
  // What the epilogue compares or rotates with comes in units, requested one ahead of their use, the first under the last MFMAs:
  // old values of a 64-column block (EPI 1), rotation factors of a 64-column block for half of the rows (EPI 2).
  constexpr int HI = EPI == 2 ? MI / 2 : MI;
  constexpr int kReq = EPI == 1 ? MI * 2 : HI * 4, kUnits = EPI == 1 ? NJ / 4 : NJ / 4 * (MI / HI);
  static_assert(EPI != 2 || MI % 2 == 0, "halves");
  // a lane's 16-byte pieces of a row (see `piece`) start here in a block of 32 columns
  const int pc = (lg & 1) * 16 + (lg >> 1) * 8;
  uint4 old[2][EPI == 1 ? MI : 1][2];
  float4 cs[2][EPI == 2 ? HI : 1][4];
  auto request = [&](int u, int q) {
    if constexpr (EPI == 1) {
      const int i = q / 2, c = crow[i] < 0 ? 0 : crow[i];  // (rows that are not scored: all the same one)
      old[u % 2][i][q % 2] = *reinterpret_cast<const uint4*>(ep->cache + static_cast<size_t>(c) * N + n0 +
                                                             (wn * (NJ / 4) + u) * 64 + q % 2 * 32 + pc);
    } else if constexpr (EPI == 2) {
      const int i = u % 2 * HI + q / 4, t0 = (wn * (NJ / 4) + u / 2) % 2 * 32 + lg * 4;
      cs[u % 2][q / 4][q % 4] =
          *reinterpret_cast<const float4*>(ep->tab + static_cast<size_t>(meta[i]) * 64 + t0 + q % 4 / 2 * 16 + q % 2 * 2);
    }
  };
  // Four columns each of blocks j (a) and j + 1 (b): lanes 16 apart trade, so that the even 16 lanes hold eight neighbouring columns of
  // j, the odd ones of j + 1.
  auto piece = [](uint2 a, uint2 b) {
    const auto x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    return make_uint4(x[0], y[0], x[1], y[1]);
  };
  int sa = 0, sb = 0;          // slots of A(kt) and B(kt)
  int sy = DY - 1;             // slot of Y(kt - 1)
  // Step kt with `left` steps to come (DX: that many or more): what would lie beyond the last block is not loaded, and of what a
  // wavefront issued last, from the end Y, X, Y, ..., only the blocks after kt + 1 may be in flight across the barrier.
  auto step = [&](int kt, auto left_) {
    constexpr int left = decltype(left_)::value;
    constexpr int kFly = left == 0 ? 0 : (DX - 2 < left - 1 ? DX - 2 : left - 1) * LX + (DY - 2 < left - 1 ? DY - 2 : left - 1) * LY;
    const int sa1 = sa + 1 < DA ? sa + 1 : 0, sb1 = sb + 1 < DB ? sb + 1 : 0;
    const int ky = left >= DY - 1 ? kof(kt + DY - 1) : 0, kx = left >= DX ? kof(kt + DX) : 0;
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    half(std::integral_constant<int, 0>{}, [&](int t) {
#pragma unroll
      for (int q = 0; q < MI + NJ; ++q)
        if (1 + q * kSpan / (MI + NJ) == t) read(sa, sb, 1, q);
#pragma unroll
      for (int l = 0; l < LY; ++l)
        if (left >= DY - 1 && l * kSpan / LY == t) issue_y(sy, ky, l);
    });
    wait_vmcnt_lds<kFly>();
    if (left > 0) __builtin_amdgcn_s_barrier();
    half(std::integral_constant<int, 1>{}, [&](int t) {
#pragma unroll
      for (int q = 0; q < MI + NJ; ++q)
        if (left > 0 && 1 + q * kSpan / (MI + NJ) == t) read(sa1, sb1, 0, q);
#pragma unroll
      for (int l = 0; l < LX; ++l)
        if (left >= DX && l * kSpan / LX == t) issue_x(XB ? sb : sa, kx, l);
      if constexpr (EPI != 0 && left == 0) {
#pragma unroll
        for (int q = 0; q < kReq; ++q)
          if (q * kSpan / kReq == t) request(0, q);
      }
    });
    sy = XB ? sa : sb;
    sa = sa1;
    sb = sb1;
  };
  int kt = 0;
  for (; kt < nkt - DX; ++kt) step(kt, std::integral_constant<int, DX>{});
  if constexpr (DX > 4) { if (nkt - kt > 4) step(kt++, std::integral_constant<int, 4>{}); }
  if constexpr (DX > 3) { if (nkt - kt > 3) step(kt++, std::integral_constant<int, 3>{}); }
  if constexpr (DX > 2) { if (nkt - kt > 2) step(kt++, std::integral_constant<int, 2>{}); }
  if (nkt - kt > 1) step(kt++, std::integral_constant<int, 1>{});
  step(kt, std::integral_constant<int, 0>{});
  // (results leave the accumulation registers behind the last wait: without this some did between the last MFMAs)
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+a"(acc[i][j]));
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (EPI == 1) {
    const int n_ct = N / 64;
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const int wv = wn * (NJ / 4) + u, ct = col_tile * (BN / 64) + wv;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        bf16_t* dst = ep->cache + static_cast<size_t>(crow[i] < 0 ? ~crow[i] : crow[i]) * N + n0 + wv * 64 + pc;
        float dot = 0.f, nn = 0.f, no = 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4 v0 = acc[i][4 * u + 2 * j], v1 = acc[i][4 * u + 2 * j + 1];
          const uint4 nv = piece(make_uint2(pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3])),
                                 make_uint2(pack_bf16x2(v1[0], v1[1]), pack_bf16x2(v1[2], v1[3])));
          if (ep->part != nullptr) {  // uniform
            const uint4 ov = old[u % 2][i][j];
            const uint32_t nw[4] = {nv.x, nv.y, nv.z, nv.w}, ow[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const float a0 = __uint_as_float(nw[t] << 16), a1 = __uint_as_float(nw[t] & 0xffff0000u);
              const float b0 = __uint_as_float(ow[t] << 16), b1 = __uint_as_float(ow[t] & 0xffff0000u);
              if (ep->metric == 0) {
                dot += a0 * b0; nn += a0 * a0; no += b0 * b0;
                dot += a1 * b1; nn += a1 * a1; no += b1 * b1;
              } else {
                const float d0 = a0 - b0, d1 = a1 - b1;
                dot += d0 * d0;
                dot += d1 * d1;
              }
            }
          }
          if (row_of(i) < M) *reinterpret_cast<uint4*>(dst + j * 32) = nv;
          if (u + 1 < kUnits) request(u + 1, 2 * i + j);
        }
        if (ep->part != nullptr) {
#pragma unroll
          for (int o = 16; o < 64; o <<= 1) {
            dot += __shfl_xor(dot, o, 64); nn += __shfl_xor(nn, o, 64); no += __shfl_xor(no, o, 64);
          }
          if (crow[i] >= 0 && lg == 0) {
            const int m = row_of(i), at = m / ep->per_seq * (ep->n - ep->L_p) + ep->first + m % ep->per_seq - ep->L_p;
            ep->part[(static_cast<size_t>(0) * n_ct + ct) * ep->part_stride + at] = dot;
            ep->part[(static_cast<size_t>(1) * n_ct + ct) * ep->part_stride + at] = nn;
            ep->part[(static_cast<size_t>(2) * n_ct + ct) * ep->part_stride + at] = no;
          }
        }
      }
    }
  } else if constexpr (EPI == 2) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      if (u + 1 < kUnits) {
#pragma unroll
        for (int q = 0; q < kReq; ++q) request(u + 1, q);
      }
      const int jh = u / 2, wv = wn * (NJ / 4) + jh;
      const int head0 = n0 + (wv / 2) * 128;  // first column of the head in [W0; W1]
      const bool is_q = head0 < N0, rotate = is_q || ep->rope_second != 0;
#pragma unroll
      for (int q = 0; q < HI; ++q) {
        const int i = u % 2 * HI + q;
        bf16_t* dst = (is_q ? ep->q_out + static_cast<size_t>(row_of(i)) * N0 + head0
                            : ep->cache + static_cast<size_t>(crow[i]) * ep->d_kv + (head0 - N0)) + (wv % 2) * 32 + pc;
        uint2 lo[2], hi[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x4 x0 = acc[i][4 * jh + j], x1 = acc[i][4 * jh + j + 2];
          if (rotate) {
            const float4 f0 = cs[u % 2][q][2 * j], f1 = cs[u % 2][q][2 * j + 1];
            const float c[4] = {f0.x, f0.z, f1.x, f1.z}, sn[4] = {f0.y, f0.w, f1.y, f1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float a = x0[e], b = x1[e];
              x0[e] = a * c[e] - b * sn[e];
              x1[e] = b * c[e] + a * sn[e];
            }
          }
          lo[j] = make_uint2(pack_bf16x2(x0[0], x0[1]), pack_bf16x2(x0[2], x0[3]));
          hi[j] = make_uint2(pack_bf16x2(x1[0], x1[1]), pack_bf16x2(x1[2], x1[3]));
        }
        const uint4 l4 = piece(lo[0], lo[1]), h4 = piece(hi[0], hi[1]);
        if (row_of(i) < M) {
          *reinterpret_cast<uint4*>(dst) = l4;
          *reinterpret_cast<uint4*>(dst + 64) = h4;
        }
      }
    }
  } else if constexpr (PAIR) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      bf16_t* dst = U + static_cast<size_t>(row_of(i)) * N + n0 + wn * (NJ / 2 * 16) + lg * 4;
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) {
        const f32x4 g = acc[i][j], up = acc[i][j + NJ / 2];
        if (row_of(i) < M)
          *reinterpret_cast<uint2*>(dst + j * 16) =
              make_uint2(pack_bf16x2(silu_mul(g[0], up[0]), silu_mul(g[1], up[1])),
                         pack_bf16x2(silu_mul(g[2], up[2]), silu_mul(g[3], up[3])));
      }
    }
  } else {
    // A W^T: a lane holds four rows of one column, 16 neighbouring lanes store 64 contiguous bytes
    float* Cs = C + static_cast<size_t>(blockIdx.z) * M * N + n0 + wn * (NJ * 16) + ln;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * (MI * 16) + i * 16 + lg * 4 + e;
        if (m < M) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) Cs[static_cast<size_t>(m) * N + j * 16] = acc[i][j][e];
        }
      }
  }
}

}  // namespace
}  // namespace dllmc
