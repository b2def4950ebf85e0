// Bidirectional softmax attention of the recomputed query rows over ALL n cached keys and
// values of their sequence, no mask (paper complexity appendix: the 4*r^*n*d term; on refresh
// steps the query set is the whole response or the whole sequence).
//
// Queries arrive compact: sequence b owns rows [b*Mq, (b+1)*Mq) of q and out.
//
//  * k_attn_simple -- any storage type / head width: one wavefront per (query, head), scores
//                     kept in LDS, two passes.  Head widths other than 64 and 128.
//  * k_attn_f32    -- float32 models with head width 64 or 128, bf16 with head width 64: float32
//                     products on the matrix cores.
//  * k_attn_mfma / k_attn_walk -- bf16, head width 128.  Flash-style online softmax on
//                     v_mfma_f32_16x16x32_bf16.  The score tile is computed transposed
//                     (S^T = K * Q^T) so that each lane ends up holding, for one query, eight
//                     keys of a 32-key block: exactly the B-operand layout of the second
//                     product O^T = V^T * P^T, so probabilities never leave registers.
//                     V tiles are transposed once per workgroup through LDS and shared by
//                     its four 16-query wavefronts.  k_attn_mfma: key ranges of up to three
//                     blocks (all of it fetched into registers before the first use), the
//                     key range split over workgroups and the partial results combined in
//                     key-range order by k_attn_merge; k_attn_walk: whole key ranges (K and V
//                     tiles staged global -> LDS several blocks ahead).
//  * k_attn_few    -- fewer than 128 queries where neither of those is the better one: the
//                     wavefronts of a workgroup split its key range.
//  * k_attn_tile   -- from 128 queries on.
#include "common.hpp"

namespace dllmc {


namespace {

template <typename T>
__global__ __launch_bounds__(64) void k_attn_simple(const T* __restrict__ q, int Mq,
                                                    const T* __restrict__ kc,
                                                    const T* __restrict__ vc, int n, int H_q,
                                                    int H_kv, int d_h, T* __restrict__ out,
                                                    const int* __restrict__ rmap) {
  extern __shared__ float sm[];
  float* qs = sm;        // [d_h]
  float* sc = sm + d_h;  // [n]
  const int i = blockIdx.x, a = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x;
  const int d_q = H_q * d_h, d_kv = H_kv * d_h;
  const int kv = a / (H_q / H_kv);
  const T* qr = q + (static_cast<size_t>(b) * Mq + i) * d_q + a * d_h;
  // row j of this sequence in the cache tensors (the row map's entry in the paged layout)
  auto crow = [&](int j) { return static_cast<size_t>(rmap ? rmap[b * n + j] : b * n + j); };
  const T* K = kc + kv * d_h;
  const T* V = vc + kv * d_h;
  const float scale = 1.0f / sqrtf(static_cast<float>(d_h));
  for (int t = lane; t < d_h; t += 64) qs[t] = ldf(qr + t);
  __syncthreads();
  float mx = -INFINITY;
  for (int j = lane; j < n; j += 64) {
    const T* kr = K + crow(j) * d_kv;
    float acc = 0.f;
    for (int t = 0; t < d_h; ++t) acc = fmaf(qs[t], ldf(kr + t), acc);
    acc *= scale;
    sc[j] = acc;
    mx = fmaxf(mx, acc);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int j = lane; j < n; j += 64) {
    const float p = expf(sc[j] - mx);
    sc[j] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  __syncthreads();
  T* o = out + (static_cast<size_t>(b) * Mq + i) * d_q + a * d_h;
  for (int t = lane; t < d_h; t += 64) {
    float acc = 0.f;
    for (int j = 0; j < n; ++j) acc = fmaf(sc[j], ldf(V + crow(j) * d_kv + t), acc);
    stf(o + t, acc / sum);
  }
}

// ---- float32 arithmetic on the matrix cores ----------------------------------------------
// k_attn_f32: float32 models with head width 64 or 128, and bf16 ones with head width 64 (converted as
// they are multiplied): products, probabilities and sums in float32, v_mfma_f32_16x16x4_f32.
// A workgroup is 16 queries of one head; its four wavefronts take a quarter of the keys each, 16 at a
// time, and their (O, m, l) meet in LDS.  As in the bf16 kernels the scores are computed transposed
// (S^T = K Q^T), so that a lane holds four keys of one query, 4 * lg .. + 3, and the product O^T = V^T
// P^T takes them as they are: instruction j multiplies the keys {4 * lg + j}.  The rows of V^T are dealt to the
// instructions' 16 rows in runs (row r of block db is dim r * D/16 + db), so that a lane's share of a
// key, and of the result, is one contiguous piece.  No LDS on the way in: an instruction takes 32 cycles
// and feeds on 4 bytes a lane.
// Bound by those instructions (2048 cycles per 16 keys and 16 queries at width 128) once there are ~256
// workgroups, by trips to memory below.  Against k_attn_simple (one wavefront per query and head, keys as
// lanes: every lane walks its own row), us: 8 queries, 96 keys, 4 heads of 64: 12.5 -> 4.6; 2 x 176
// queries, 176 keys, 8 heads of 128: 73.6 -> 9.4.
template <typename T> struct Quad;  // four neighbouring elements as loaded, and as float32
template <> struct Quad<float> {
  typedef f32x4 raw;
  static __device__ __forceinline__ f32x4 f32(const raw& r) { return r; }
};
template <> struct Quad<bf16_t> {
  typedef uint2 raw;
  static __device__ __forceinline__ f32x4 f32(const raw& r) {
    return f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                 __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
  }
};

constexpr int kFW = 4;  // wavefronts of a workgroup: parts of the key range

template <typename T, int D, bool PAGED>
__global__ __launch_bounds__(64 * kFW, 2) void k_attn_f32(const T* __restrict__ q, int Mq,
                                                          const T* __restrict__ kc,
                                                          const T* __restrict__ vc, int n, int H_q,
                                                          int H_kv, T* __restrict__ out,
                                                          const int* __restrict__ rmap) {
  constexpr int C = D / 16;  // 16-dim blocks
  typedef typename Quad<T>::raw raw_t;
  __shared__ __attribute__((aligned(16))) float o_part[kFW][16][D + 4];
  __shared__ float m_part[kFW][16], l_part[kFW][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int ln = lane % 16, lg = lane / 16;
  const int i0 = blockIdx.x * 16, a = blockIdx.y, b = blockIdx.z;
  const int d_q = H_q * D, d_kv = H_kv * D;
  const int kv = a / (H_q / H_kv);
  const T* K = kc + kv * D + lg * 4;
  const T* V = vc + kv * D + ln * C;
  const int seq0 = b * n;

  // Q fragments: query ln, dims 16c + 4lg .. + 3 (queries past the end repeat the last one, never stored)
  f32x4 qf[C];
  {
    const T* qr = q + (static_cast<size_t>(b) * Mq + min(i0 + ln, Mq - 1)) * d_q + a * D + lg * 4;
#pragma unroll
    for (int c = 0; c < C; ++c) qf[c] = Quad<T>::f32(*reinterpret_cast<const raw_t*>(qr + c * 16));
  }
  const float scale = 1.0f / sqrtf(static_cast<float>(D));
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o_acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o_acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nblk = (n + 15) / 16;
  const int per = (nblk + kFW - 1) / kFW;
  const int blk0 = min(wave * per, nblk), blk1 = min(nblk, blk0 + per);

  struct Block { raw_t k[C], v[4][C / 4]; };
  // keys past the end repeat the last one and are masked; blocks past the range repeat its last one
  auto fetch = [&](int blk, Block& t) {
    const int key0 = min(blk, blk1 - 1) * 16;
    auto row = [&](int key) {
      const int r = seq0 + min(key, n - 1);
      return static_cast<size_t>(PAGED ? rmap[r] : r) * d_kv;
    };
    const T* kr = K + row(key0 + ln);
#pragma unroll
    for (int c = 0; c < C; ++c) t.k[c] = *reinterpret_cast<const raw_t*>(kr + c * 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const T* vr = V + row(key0 + 4 * lg + j);
#pragma unroll
      for (int c = 0; c < C / 4; ++c) t.v[j][c] = *reinterpret_cast<const raw_t*>(vr + c * 4);
    }
  };
  auto use = [&](int blk, Block& t) {
    f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;  // (two chains: an instruction may not wait for its predecessor)
#pragma unroll
    for (int c = 0; c < C; c += 2) {
      const f32x4 k0 = Quad<T>::f32(t.k[c]), k1 = Quad<T>::f32(t.k[c + 1]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k0[e], qf[c][e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k1[e], qf[c + 1][e], s1, 0, 0, 0);
      }
    }
    float p[4];
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = blk * 16 + 4 * lg + e < n ? (s0[e] + s1[e]) * scale : -INFINITY;
      mx = fmaxf(mx, p[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
      const float alpha = expf(m_run - m_use);  // 0 while nothing has been seen yet
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int c = 0; c < C; ++c) o_acc[c] *= alpha;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = expf(p[e] - m_use);
      l_run += p[e];
    }
    // The values of masked keys do not count, not even an infinity times 0.  (40 queries, 1001 keys, 8 heads of 128:
    // 28.0 us without this, 28.9 with it; selects in the product 31.4, a row of zeros to load instead 35.7, the last
    // block as a variant of its own 29.7.)
    if (blk * 16 + 16 > n) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (blk * 16 + 4 * lg + j >= n) {
#pragma unroll
          for (int c = 0; c < C / 4; ++c) t.v[j][c] = raw_t{};
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < C / 4; ++c) {
        const f32x4 v = Quad<T>::f32(t.v[j][c]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o_acc[4 * c + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], p[j], o_acc[4 * c + e], 0, 0, 0);
      }
  };
  if (blk0 < blk1) {
    Block b0, b1;  // two register sets that swap roles: the next block is in flight under this one
    fetch(blk0, b0);
    int blk = blk0;
    for (; blk + 1 < blk1; blk += 2) {
      fetch(blk + 1, b1);
      use(blk, b0);
      fetch(blk + 2, b0);
      use(blk + 1, b1);
    }
    if (blk < blk1) use(blk, b0);
  }
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);

  // lane: query ln, dims (4lg + i) * C + 0 .. C - 1
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < C; c += 4)
      *reinterpret_cast<float4*>(&o_part[wave][ln][(4 * lg + i) * C + c]) =
          make_float4(o_acc[c][i], o_acc[c + 1][i], o_acc[c + 2][i], o_acc[c + 3][i]);
  if (lg == 0) {
    m_part[wave][ln] = m_run;
    l_part[wave][ln] = l_run;
  }
  __syncthreads();
  // 16 threads per query, D / 16 dims each; the parts in key order
  const int qi = threadIdx.x / 16, t = threadIdx.x % 16;
  if (i0 + qi >= Mq) return;
  float M = m_part[0][qi];
#pragma unroll
  for (int w = 1; w < kFW; ++w) M = fmaxf(M, m_part[w][qi]);
  float L = 0.f, o[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o[c] = 0.f;
#pragma unroll
  for (int w = 0; w < kFW; ++w) {
    const float mw = m_part[w][qi];
    const float f = mw == -INFINITY ? 0.f : expf(mw - M);
    L += l_part[w][qi] * f;
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] += o_part[w][qi][c * 16 + t] * f;
  }
  T* dst = out + (static_cast<size_t>(b) * Mq + i0 + qi) * d_q + a * D;
#pragma unroll
  for (int c = 0; c < C; ++c) stf(dst + c * 16 + t, o[c] / L);
}

constexpr int kDH = 128;       // head width of the bf16 MFMA kernels
constexpr int kVtStride = 40;  // 32 keys + 8 pad (bf16 elements) per transposed V row
constexpr int kQT = 64;        // queries per workgroup: four wavefronts x 16
constexpr int kPreload = 3;    // key ranges of up to this many 32-key blocks are fetched whole
constexpr int kMaxKeySplit = 16;

// One 32-key block for a wavefront's 16 queries: scores S^T = K Q^T, running softmax (base 2),
// O^T += V^T P^T.  kf: K fragments (lane: key sb*16 + ln, dims 32c + 8lg .. +8); qf: Q fragments
// (lane: query ln, same dims); vt: the block's V tile transposed, [dim][VS keys] (SWZ: with the
// key pairs of a row permuted, see k_attn_mfma).
template <int VS, bool SWZ>
__device__ __forceinline__ void attn_block(const bf16x8 (&kf)[2][4], const bf16x8 (&qf)[4],
                                           const bf16_t* vt, int key0, int n, int ln, int lg,
                                           float sl2e, float& m_run, float& l_run,
                                           f32x4 (&o_acc)[8]) {
  f32x4 st[2];
#pragma unroll
  for (int sb = 0; sb < 2; ++sb) {
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[sb][c], qf[c], acc, 0, 0, 0);
    st[sb] = acc;
  }
  // lane holds keys key0 + sb*16 + 4*lg + i of query ln
  float p[8];
  float mx = -INFINITY;
  if (key0 + 32 <= n) {  // the whole block lies inside the sequence (wavefront-uniform)
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[sb * 4 + i] = st[sb][i];
        mx = fmaxf(mx, st[sb][i]);
      }
  } else {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = key0 + sb * 16 + 4 * lg + i;
        const float v = key < n ? st[sb][i] : -INFINITY;
        p[sb * 4 + i] = v;
        mx = fmaxf(mx, v);
      }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  // running maximum of the scaled scores (the scale is positive, so it commutes with the max)
  const float m_new = fmaxf(m_run, mx * sl2e);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  // The accumulators are rescaled only in the blocks in which some query's maximum moved
  // (wavefront-uniform test): with alpha == 1 for every lane the multiplications change nothing.
  if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);  // 0 while nothing has been seen yet
    l_run *= alpha;
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      o_acc[db][0] *= alpha;
      o_acc[db][1] *= alpha;
      o_acc[db][2] *= alpha;
      o_acc[db][3] *= alpha;
    }
  }
  // probabilities as a bf16 pair (high part + remainder): the second product then carries
  // ~16 bits of each probability instead of 8
  // (the hardware's 2^x as it is: the arguments are <= 0, and results below the normal range, which
  // it flushes to zero, are far below anything a bf16 pair can carry)
  float psum = 0.f;
  bf16x8 pf, pl;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    const float e0 = __builtin_amdgcn_exp2f(fmaf(p[t], sl2e, -m_use));
    const float e1 = __builtin_amdgcn_exp2f(fmaf(p[t + 1], sl2e, -m_use));
    psum += e0;
    psum += e1;
    const uint32_t hi = pack_bf16x2(e0, e1);
    reinterpret_cast<uint32_t*>(&pf)[t / 2] = hi;
    reinterpret_cast<uint32_t*>(&pl)[t / 2] =
        pack_bf16x2(e0 - __uint_as_float(hi << 16), e1 - __uint_as_float(hi & 0xffff0000u));
  }
  l_run += psum;
  // O^T[dim][query] += V^T[dim][key] * P^T[key][query]
#pragma unroll
  for (int db = 0; db < 8; ++db) {
    // SWZ: key pair p of the rows of dim block db sits at pair position p ^ 2*db
    const bf16_t* vrow = vt + (db * 16 + ln) * VS;
    const uint2 lo = *reinterpret_cast<const uint2*>(vrow + (SWZ ? (4 * lg) ^ (4 * db) : 4 * lg));
    const uint2 hi =
        *reinterpret_cast<const uint2*>(vrow + (SWZ ? (16 + 4 * lg) ^ (4 * db) : 16 + 4 * lg));
    const uint4 both = make_uint4(lo.x, lo.y, hi.x, hi.y);
    const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
    o_acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o_acc[db], 0, 0, 0);
    o_acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl, o_acc[db], 0, 0, 0);
  }
}

// End of a key range for query iq (lane's column of O^T): with KS == 1 the normalised output row,
// otherwise the un-normalised partial (O, m, l) of range ks for k_attn_merge.
__device__ __forceinline__ void attn_finish(const f32x4 (&o_acc)[8], float m_run, float l_run, int iq,
                                            int Mq, int b, int a, int ks, int KS, int H_q, int lg,
                                            bf16_t* __restrict__ out, float* __restrict__ part) {
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (iq >= Mq) return;
  const int d_q = H_q * kDH;
  if (KS == 1) {
    const float inv_l = 1.0f / l_run;
    bf16_t* o = out + (static_cast<size_t>(b) * Mq + iq) * d_q + a * kDH;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      uint2 t;
      t.x = static_cast<uint32_t>(f32_to_bf16(o_acc[db][0] * inv_l)) |
            (static_cast<uint32_t>(f32_to_bf16(o_acc[db][1] * inv_l)) << 16);
      t.y = static_cast<uint32_t>(f32_to_bf16(o_acc[db][2] * inv_l)) |
            (static_cast<uint32_t>(f32_to_bf16(o_acc[db][3] * inv_l)) << 16);
      *reinterpret_cast<uint2*>(o + db * 16 + 4 * lg) = t;
    }
  } else {
    // part[((b*Mq + iq)*H_q + a)*KS + ks][kDH + 2]
    float* w = part + ((static_cast<size_t>(b) * Mq + iq) * H_q + a) * KS * (kDH + 2) +
               static_cast<size_t>(ks) * (kDH + 2);
#pragma unroll
    for (int db = 0; db < 8; ++db)
      *reinterpret_cast<float4*>(w + db * 16 + 4 * lg) =
          make_float4(o_acc[db][0], o_acc[db][1], o_acc[db][2], o_acc[db][3]);
    if (lg == 0) {
      w[kDH] = m_run;
      w[kDH + 1] = l_run;
    }
  }
}

// Workgroups are handed to the 8 XCDs round-robin in launch order and each XCD has its own L2.
// The launch is one-dimensional: a "slot" is (query tile, KV head, sequence, key range), and the G
// query heads that share the slot's KV head run back to back on one XCD, so the slot's K and V
// blocks are fetched into that L2 once instead of once per query head (grouped KV heads: 7 x
// fewer fetches for 28 / 4 heads).  Slots beyond the last multiple of 8 are walked in order.
struct AttnWork { int qtile, a, b, ks; };
__device__ __forceinline__ AttnWork attn_work(int qt, int H_q, int H_kv, int KS) {
  const int G = H_q / H_kv;
  const int n_slots = gridDim.x / G;
  const int lin = blockIdx.x;
  const int n8 = n_slots & ~7;
  int slot, j;
  if (lin < n8 * G) {
    const int xcd = lin & 7, idx = lin >> 3;
    slot = (idx / G) * 8 + xcd;
    j = idx % G;
  } else {
    const int rest = lin - n8 * G;
    slot = n8 + rest / G;
    j = rest % G;
  }
  // slot = ((b * KS + ks) * H_kv + kvh) * qt + qtile
  AttnWork w;
  w.qtile = slot % qt;
  const int kvh = (slot / qt) % H_kv;
  const int z = slot / (qt * H_kv);
  w.b = z / KS;
  w.ks = z % KS;
  w.a = kvh * G + j;
  return w;
}

// Workgroup = 4 wavefronts = 4 tiles of 16 queries of one head and one sequence; the slot
// enumerates (sequence, key range).  All four wavefronts use the same 32-key blocks, so a V
// tile is transposed through LDS once per workgroup.  With KS == 1 the normalised output is
// written; otherwise the un-normalised partial (O, m, l) of this key range goes to `part` for
// k_attn_merge.
// k_attn_mfma: key ranges of at most kPreload blocks (the launcher guarantees it: split keys of
// an adaptive step).  Every K fragment and V tile of the range is requested before the first
// one is used, so the range costs one trip to memory instead of one per block.
// V transposition: thread = (key pair kp, 16-byte chunk ch) loads the chunk of keys 2kp and 2kp+1
// (16 consecutive lanes read one key's 256 bytes) and writes, per dim, one 32-bit word holding
// both keys at pair position kp ^ (ch & 14) of the dim's row: the 16 lanes of a key pair then
// hit 16 different banks (lanes along the dims with 16-bit stores spend 7 of 8 LDS cycles on
// bank conflicts), and ch & 14 = 2 * (dim / 16) is the same for all rows of a dim block, so the
// reader undoes it with a constant.
// PAGED: the key rows are looked up in the row map (a compile-time switch: the flat layout's
// code, whose loads must all go out before the first use, stays exactly as it is without it).
template <bool PAGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_attn_mfma(
    const bf16_t* __restrict__ q, int Mq, const bf16_t* __restrict__ kc,
    const bf16_t* __restrict__ vc, int n, int H_q, int H_kv, int KS, bf16_t* __restrict__ out,
    float* __restrict__ part, const int* __restrict__ rmap) {
  __shared__ __attribute__((aligned(16))) bf16_t Vt[kPreload][kDH * kVtStride];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;  // scalar
  const int ln = lane % 16, lg = lane / 16;
  const AttnWork wk = attn_work((Mq + kQT - 1) / kQT, H_q, H_kv, KS);
  const int a = wk.a, b = wk.b, ks = wk.ks;
  const int d_q = H_q * kDH, d_kv = H_kv * kDH;
  const int kv = a / (H_q / H_kv);
  const int i0 = wk.qtile * kQT + wave * 16;  // first query of this wavefront

  // key row j of this sequence: cache row b * n + j, or the row map's entry (paged layout)
  const bf16_t* K = kc + kv * kDH;
  const bf16_t* V = vc + kv * kDH;
  const int seq0 = b * n;

  // Q fragments (B operand of S^T = K Q^T): lane (query ln, group lg) holds dims 32c+8lg..+8
  int qi = i0 + ln;
  if (qi >= Mq) qi = Mq - 1;  // padded queries compute a duplicate that is never stored
  const bf16_t* qr = q + (static_cast<size_t>(b) * Mq + qi) * d_q + a * kDH + lg * 8;
  bf16x8 qf[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) qf[c] = *reinterpret_cast<const bf16x8*>(qr + c * 32);

  const float sl2e = 1.4426950408889634f / sqrtf(static_cast<float>(kDH));  // scale * log2(e)
  float m_run = -INFINITY;  // running maximum of the scaled scores (base 2), per query
  float l_run = 0.f;        // this lane's share of the running denominator
  f32x4 o_acc[8];           // O^T: dims db*16 + 4*lg + i, query ln
#pragma unroll
  for (int db = 0; db < 8; ++db) o_acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nblk = (n + 31) / 32;
  const int per = (nblk + KS - 1) / KS;
  const int blk0 = ks * per;
  const int blk1 = min(nblk, blk0 + per);
  const int nb = blk1 - blk0;

  if (nb > 0) {
    const int kp = threadIdx.x / 16, ch = threadIdx.x % 16;
    bf16x8 kall[kPreload][2][4];
    uint4 vall[kPreload][2];
#pragma unroll
    for (int j = 0; j < kPreload; ++j) {
      const int blk = min(blk0 + j, blk1 - 1);  // blocks past the range repeat the last one, unused
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        int kr = blk * 32 + sb * 16 + ln;
        if (kr >= n) kr = n - 1;  // masked in the scores; any finite value will do
        const size_t cr = static_cast<size_t>(PAGED ? rmap[seq0 + kr] : seq0 + kr);
        const bf16_t* kptr = K + cr * d_kv + lg * 8;
#pragma unroll
        for (int c = 0; c < 4; ++c) kall[j][sb][c] = *reinterpret_cast<const bf16x8*>(kptr + c * 32);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int kr = blk * 32 + 2 * kp + h;
        if (kr >= n) kr = n - 1;
        const size_t cr = static_cast<size_t>(PAGED ? rmap[seq0 + kr] : seq0 + kr);
        vall[j][h] = *reinterpret_cast<const uint4*>(V + cr * d_kv + ch * 8);
      }
    }
#pragma unroll
    for (int j = 0; j < kPreload; ++j) {
      uint32_t* vt32 = reinterpret_cast<uint32_t*>(Vt[j]);
      const uint32_t e0[4] = {vall[j][0].x, vall[j][0].y, vall[j][0].z, vall[j][0].w};
      const uint32_t e1[4] = {vall[j][1].x, vall[j][1].y, vall[j][1].z, vall[j][1].w};
      const int pos = kp ^ (ch & 14);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int dim = ch * 8 + 2 * t;
        vt32[(dim * kVtStride) / 2 + pos] = (e0[t] & 0xffffu) | (e1[t] << 16);
        vt32[((dim + 1) * kVtStride) / 2 + pos] = (e0[t] >> 16) | (e1[t] & 0xffff0000u);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreload; ++j)
      if (j < nb)
        attn_block<kVtStride, true>(kall[j], qf, Vt[j], (blk0 + j) * 32, n, ln, lg, sl2e, m_run, l_run,
                                    o_acc);
  }
  attn_finish(o_acc, m_run, l_run, i0 + ln, Mq, b, a, ks, KS, H_q, lg, out, part);
}

// ---- long key ranges -----------------------------------------------------------------
// k_attn_walk: the same tiling and arithmetic as k_attn_mfma for all keys of a sequence (enough
// workgroups to fill the chip without splitting them).  A block-by-block walk that fetches one block ahead
// into registers is bound by the memory latency of every block; here the K and V tiles of a
// block go from global memory straight into LDS (global_load_lds: no registers held while they
// are in flight), kWalkStages - 1 blocks ahead.  K fragments are then read from LDS (slot =
// chunk ^ (key % 16), so the 16 keys of a fragment read hit 16 different slots); the V tile is
// read back row-wise and written transposed into Vt as in the other kernel.
constexpr int kWalkStages = 4;
constexpr int kVtStrideW = 36;  // 32 keys + 4 pad: rows of 8 dims apart start 16 banks apart

// (The body is a function of its own with restrict-qualified parameters, inlined into the kernel:
// only then does the compiler keep the global -> LDS loads of the later stages in flight across
// the LDS reads of the landed one; written directly into the kernel it waits for every load in
// flight before each of those reads, and the walk is bound by one memory latency per block.  The
// waits that order the loads against the reads are the explicit ones below.)
template <bool PAGED>
__device__ __forceinline__ void attn_walk_body(const bf16_t* __restrict__ q, int Mq,
                                               const bf16_t* __restrict__ kc,
                                               const bf16_t* __restrict__ vc, int n, int H_q,
                                               int H_kv, bf16_t* __restrict__ out,
                                               const int* __restrict__ rmap) {
  // [stage][K tile, V tile][32 keys][16 slots of 16 bytes], then the transposed V tile.  One LDS
  // object on purpose: with two, the compiler cannot tell reads of the landed stage from the
  // loads in flight into the other stages and waits for all of those before every read.
  constexpr int kTileVecs = kWalkStages * 2 * 32 * 16;
  __shared__ __attribute__((aligned(1024))) uint4 smem[kTileVecs + kDH * kVtStrideW * 2 / 16];
  uint4 (*tiles)[2][32 * 16] = reinterpret_cast<uint4 (*)[2][32 * 16]>(smem);
  bf16_t* Vt = reinterpret_cast<bf16_t*>(smem + kTileVecs);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;  // scalar
  const int ln = lane % 16, lg = lane / 16;
  const AttnWork wk = attn_work((Mq + kQT - 1) / kQT, H_q, H_kv, 1);
  const int a = wk.a, b = wk.b;
  const int d_q = H_q * kDH, d_kv = H_kv * kDH;
  const int kv = a / (H_q / H_kv);
  const int i0 = wk.qtile * kQT + wave * 16;

  const bf16_t* K = kc + kv * kDH;
  const bf16_t* V = vc + kv * kDH;
  const int seq0 = b * n;

  int qi = i0 + ln;
  if (qi >= Mq) qi = Mq - 1;  // padded queries compute a duplicate that is never stored
  const bf16_t* qr = q + (static_cast<size_t>(b) * Mq + qi) * d_q + a * kDH + lg * 8;
  bf16x8 qf[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) qf[c] = *reinterpret_cast<const bf16x8*>(qr + c * 32);

  const float sl2e = 1.4426950408889634f / sqrtf(static_cast<float>(kDH));
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o_acc[8];
#pragma unroll
  for (int db = 0; db < 8; ++db) o_acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nb = (n + 31) / 32;
  // loader: a tile is 8 wavefront instructions of 4 keys x 256 bytes; wavefront w issues
  // instructions 2w and 2w+1 of the K and of the V tile.  Lane l: key 4q + l/16, slot l%16.
  // LDS slot l%16 of a key's row holds chunk slot ^ (key % 16) of K (the 16 keys of a
  // fragment read hit 16 slots) and chunk slot ^ (key/2 % 16) of V (so do the 16 key pairs
  // of the transposition)
  int lkey[2], kchunk[2], vchunk[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    lkey[j] = 4 * (2 * wave + j) + lane / 16;
    kchunk[j] = (lane % 16) ^ (lkey[j] % 16);
    vchunk[j] = (lane % 16) ^ ((lkey[j] >> 1) % 16);
  }
  // cache rows of this lane's two keys of a block: the rows themselves, or (paged layout) the
  // row map's entries, looked up one block before the block's loads are issued
  auto rows_of = [&](int blk, int (&cr)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int kr = blk * 32 + lkey[j];
      if (kr >= n) kr = n - 1;  // masked in the scores; any finite value will do
      cr[j] = PAGED ? rmap[seq0 + kr] : seq0 + kr;
    }
  };
  auto issue = [&](const int (&cr)[2], int stage) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const size_t row = static_cast<size_t>(cr[j]) * d_kv;
      __builtin_amdgcn_global_load_lds(K + row + kchunk[j] * 8, &tiles[stage][0][(2 * wave + j) * 64],
                                       16, 0, 0);
      __builtin_amdgcn_global_load_lds(V + row + vchunk[j] * 8, &tiles[stage][1][(2 * wave + j) * 64],
                                       16, 0, 0);
    }
  };
  // blocks past the range repeat the last one (never used): the number of loads in flight
  // stays the same in every iteration
  int cr_next[2];
#pragma unroll
  for (int s = 0; s < kWalkStages - 1; ++s) {
    rows_of(min(s, nb - 1), cr_next);
    issue(cr_next, s);
  }
  rows_of(min(kWalkStages - 1, nb - 1), cr_next);

  // V transposition: thread = (key pair kp, 16-byte chunk vch); it reads the chunk of keys 2kp
  // and 2kp+1 and writes, per dim, one 32-bit word holding both keys.  Consecutive lanes write
  // consecutive words of a Vt row and the four chunks of a wavefront sit 16 banks apart (row
  // stride 36 elements), so the writes are free of bank conflicts; 16-bit stores with lanes
  // along the dims spend 7 of 8 LDS cycles on conflicts.
  const int kp = threadIdx.x % 16, vch = threadIdx.x / 16;
  uint32_t* vt32 = reinterpret_cast<uint32_t*>(Vt);
  // (paged layout: block 0 is older than the loads of the blocks after it, wherever the compiler has put the lookups)
  if (PAGED) wait_vmcnt<4 * (kWalkStages - 2)>();
  for (int i = 0; i < nb; ++i) {
    const int stage = i % kWalkStages;
    // 4 loads per block and wavefront, kWalkStages - 1 blocks in flight: the oldest has landed
    // (paged layout: the two row-map lookups of the block after those are in flight as well)
    wait_vmcnt<4 * (kWalkStages - 2) + (PAGED ? 2 : 0)>();
    // everybody's loads of block i have landed, and everybody is done with block i - 1: its
    // stage and Vt may be overwritten
    __builtin_amdgcn_s_barrier();
    // (paged layout: the compiler waits for the lookups with vmcnt(0), see k_attn_few)
    const int cr_use[2] = {cr_next[0], cr_next[1]};
    rows_of(min(i + kWalkStages, nb - 1), cr_next);
    issue(cr_use, (i + kWalkStages - 1) % kWalkStages);
    {
      const uint4 r0 = tiles[stage][1][(2 * kp) * 16 + (vch ^ kp)];
      const uint4 r1 = tiles[stage][1][(2 * kp + 1) * 16 + (vch ^ kp)];
      const uint32_t e0[4] = {r0.x, r0.y, r0.z, r0.w}, e1[4] = {r1.x, r1.y, r1.z, r1.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int dim = vch * 8 + 2 * j;
        vt32[(dim * kVtStrideW) / 2 + kp] = (e0[j] & 0xffffu) | (e1[j] << 16);
        vt32[((dim + 1) * kVtStrideW) / 2 + kp] = (e0[j] >> 16) | (e1[j] & 0xffff0000u);
      }
    }
    // K fragments of this wavefront: key sb*16 + ln, dims 32c + 8lg .. +8 = chunk 4c + lg
    bf16x8 kf[2][4];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        kf[sb][c] = __builtin_bit_cast(bf16x8, tiles[stage][0][(sb * 16 + ln) * 16 + ((4 * c + lg) ^ ln)]);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // LDS writes of Vt done (lgkmcnt 0); global loads stay in flight
    __builtin_amdgcn_s_barrier();
    attn_block<kVtStrideW, false>(kf, qf, Vt, i * 32, n, ln, lg, sl2e, m_run, l_run, o_acc);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the repeated loads past the range, before the LDS goes away
  attn_finish(o_acc, m_run, l_run, i0 + ln, Mq, b, a, 0, 1, H_q, lg, out, nullptr);
}

template <bool PAGED>
__global__ __launch_bounds__(256) void k_attn_walk(const bf16_t* __restrict__ q, int Mq,
                                                   const bf16_t* __restrict__ kc,
                                                   const bf16_t* __restrict__ vc, int n, int H_q,
                                                   int H_kv, bf16_t* __restrict__ out,
                                                   const int* __restrict__ rmap) {
  attn_walk_body<PAGED>(q, Mq, kc, vc, n, H_q, H_kv, out, rmap);
}

// ---- many queries --------------------------------------------------------------------
// k_attn_tile: refresh steps and batched sequences, where a (sequence, head) has hundreds of
// queries and the work is bound by the matrix cores, the LDS and the softmax arithmetic rather
// than by the K/V stream.  Against k_attn_walk: a wavefront owns 32 queries (two 16-query
// column blocks), so every K and V fragment read from LDS feeds two MFMAs; blocks are 64 keys
// (one barrier per 64 keys instead of two per 32); and V is never transposed through LDS: the
// A operand of O^T += V^T P^T (lane: one dim, eight keys) comes straight out of the row-major V
// tile with ds_read_b64_tr_b16.  That instruction works on groups of 16 lanes: lane 4t + q of a
// group passes the address of four consecutive 16-bit elements -- elements 4q .. 4q+3 of row t of
// a 4 x 16 block -- and lane i of the group receives element i of rows 0..3 (layout checked on the
// hardware).  Here a group's rows are the keys 4*lg .. 4*lg+3 of a 16-key sub-block and the 16
// elements a dim block, so lane (ln, lg) gets keys 4*lg .. +3 at dim db*16 + ln: with two such reads
// (sub-blocks 2h and 2h+1) exactly the keys whose probabilities the lane holds after the first
// product.  Two LDS stages of K tile + V tile (64 KB, two workgroups per CU); the tiles arrive by
// global_load_lds with slot = chunk ^ (key % 16) for both, which keeps the K fragment reads (16
// keys, one chunk each) and the transposing reads (16 keys x 32 bytes) spread over all banks.
// Workgroup order of k_attn_tile: a "group" is everything that reads the same K and V rows -- the
// query tiles of all query heads of one KV head, for one sequence and key range.  Groups go to the
// XCDs round-robin and an XCD works through its groups one after the other, so the group's K/V
// blocks are fetched into that XCD's L2 once and then hit by its other workgroups (with the tiles
// of a head dealt over all XCDs, every XCD streams every head's keys: 2.7 GB from beyond L2 for the
// 4608-row refresh, 36 times the K/V cache).  Groups beyond the last multiple of 8 are walked in
// launch order.
__device__ __forceinline__ AttnWork attn_work_tile(int qt, int H_q, int H_kv, int KS) {
  const int G = H_q / H_kv;
  const int W = G * qt;  // workgroups per group
  const int n_groups = gridDim.x / W;
  const int lin = blockIdx.x;
  const int n8 = n_groups & ~7;
  int group, w;
  if (lin < n8 * W) {
    const int xcd = lin & 7, idx = lin >> 3;
    group = (idx / W) * 8 + xcd;
    w = idx % W;
  } else {
    const int rest = lin - n8 * W;
    group = n8 + rest / W;
    w = rest % W;
  }
  // group = (b * KS + ks) * H_kv + kvh;  w = j * qt + qtile
  AttnWork r;
  r.qtile = w % qt;
  const int kvh = group % H_kv;
  const int z = group / H_kv;
  r.b = z / KS;
  r.ks = z % KS;
  r.a = kvh * G + w / qt;
  return r;
}

constexpr int kTQ = 128;  // queries per workgroup
constexpr int kTK = 64;   // keys per block
constexpr float kLazy = 8.0f;
typedef short v4i16_t __attribute__((ext_vector_type(4)));

template <bool PAGED>
__device__ __forceinline__ void attn_tile_body(const bf16_t* __restrict__ q, int Mq,
                                               const bf16_t* __restrict__ kc,
                                               const bf16_t* __restrict__ vc, int n, int H_q,
                                               int H_kv, int KS, bf16_t* __restrict__ out,
                                               float* __restrict__ part,
                                               const int* __restrict__ rmap) {
  // [stage][K tile, V tile][64 keys][16 slots of 16 bytes]
  __shared__ __attribute__((aligned(1024))) uint4 tiles[2][2][kTK * 16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;  // scalar
  const int ln = lane % 16, lg = lane / 16;
  const AttnWork wk = attn_work_tile((Mq + kTQ - 1) / kTQ, H_q, H_kv, KS);
  const int a = wk.a, b = wk.b, ks = wk.ks;
  const int d_q = H_q * kDH, d_kv = H_kv * kDH;
  const int kv = a / (H_q / H_kv);
  const int i0 = wk.qtile * kTQ + wave * 32;  // first query of this wavefront

  const bf16_t* K = kc + kv * kDH;
  const bf16_t* V = vc + kv * kDH;
  const int seq0 = b * n;

  // Q fragments of the two query blocks: lane (query ln, group lg) holds dims 32c + 8lg .. +8
  bf16x8 qf[2][4];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    int qi = i0 + qb * 16 + ln;
    if (qi >= Mq) qi = Mq - 1;  // padded queries compute a duplicate that is never stored
    const bf16_t* qr = q + (static_cast<size_t>(b) * Mq + qi) * d_q + a * kDH + lg * 8;
#pragma unroll
    for (int c = 0; c < 4; ++c) qf[qb][c] = *reinterpret_cast<const bf16x8*>(qr + c * 32);
  }

  const float sl2e = 1.4426950408889634f / sqrtf(static_cast<float>(kDH));
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
  f32x4 o_acc[2][8];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
#pragma unroll
    for (int db = 0; db < 8; ++db) o_acc[qb][db] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nblk = (n + kTK - 1) / kTK;
  const int per = (nblk + KS - 1) / KS;
  const int blk0 = ks * per;
  const int blk1 = min(nblk, blk0 + per);
  const int nb = blk1 - blk0;

  if (nb > 0) {
    // loader: a tile is 16 wavefront instructions of 4 keys x 256 bytes; wavefront w issues
    // instructions 4w .. 4w+3 of the K and of the V tile.  Lane l: key 4q + l/16, slot l%16.
    int lkey[4], chunk[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lkey[j] = 4 * (4 * wave + j) + lane / 16;
      chunk[j] = (lane % 16) ^ (lkey[j] % 16);
    }
    auto rows_of = [&](int blk, int (&cr)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int kr = blk * kTK + lkey[j];
        if (kr >= n) kr = n - 1;  // masked in the scores; any finite value will do
        cr[j] = PAGED ? rmap[seq0 + kr] : seq0 + kr;
      }
    };
    auto issue = [&](const int (&cr)[4], int stage) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const size_t row = static_cast<size_t>(cr[j]) * d_kv;
        __builtin_amdgcn_global_load_lds(K + row + chunk[j] * 8, &tiles[stage][0][(4 * wave + j) * 64], 16,
                                         0, 0);
        __builtin_amdgcn_global_load_lds(V + row + chunk[j] * 8, &tiles[stage][1][(4 * wave + j) * 64], 16,
                                         0, 0);
      }
    };
    // flat layout: a block's rows are 64 rows further on than the previous block's, so the loads
    // take fixed per-lane pointers plus one scalar offset (a block that sticks out of the sequence
    // goes the general way, with its rows clamped)
    const bf16_t* kbase[4];
    const bf16_t* vbase[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const size_t row = static_cast<size_t>(seq0 + blk0 * kTK + lkey[j]) * d_kv;  // may lie past the end: unused then
      kbase[j] = K + row + chunk[j] * 8;
      vbase[j] = V + row + chunk[j] * 8;
    }
    auto issue_block = [&](int blk, const int (&cr)[4], int stage) {
      if (PAGED || (blk + 1) * kTK > n) {
        issue(cr, stage);
      } else {
        const size_t off = static_cast<size_t>(blk - blk0) * kTK * d_kv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          __builtin_amdgcn_global_load_lds(kbase[j] + off, &tiles[stage][0][(4 * wave + j) * 64], 16, 0, 0);
          __builtin_amdgcn_global_load_lds(vbase[j] + off, &tiles[stage][1][(4 * wave + j) * 64], 16, 0, 0);
        }
      }
    };
    int cr_next[4];
    rows_of(blk0, cr_next);
    issue_block(blk0, cr_next, 0);
    rows_of(min(blk0 + 1, blk1 - 1), cr_next);

    // transposing reads: as lane 4t + q of its group this lane names key row 4*lg + t of a 16-key
    // sub-block and dims 4q .. 4q+3 of a dim block; byte offset inside a V tile for dim block db,
    // sub-block 0 (a sub-block further on is 16 rows = 4096 bytes further)
    const int tt = ln / 4, tq = ln % 4;
    const int krow = 4 * lg + tt;  // = key % 16
    int voff[8];
#pragma unroll
    for (int db = 0; db < 8; ++db)
      voff[db] = (krow * 16 + ((2 * db + tq / 2) ^ krow)) * 16 + (tq % 2) * 8;

    for (int i = 0; i < nb; ++i) {
      const int stage = i & 1;
      // this wavefront's loads of block i have landed and its LDS reads of block i - 1 are
      // complete; behind the barrier that holds for everybody, and the other stage is free
      wait_vmcnt_lds<0>();
      __builtin_amdgcn_s_barrier();
      if (i + 1 < nb) {
        const int cr_use[4] = {cr_next[0], cr_next[1], cr_next[2], cr_next[3]};
        issue_block(blk0 + i + 1, cr_use, stage ^ 1);
        rows_of(min(blk0 + i + 2, blk1 - 1), cr_next);
      }
      const uint4* kt = tiles[stage][0];
      const char* vt = reinterpret_cast<const char*>(tiles[stage][1]);
      const int key0 = (blk0 + i) * kTK;
      // scores S^T = K Q^T: lane holds keys key0 + sb*16 + 4*lg + e of query ln (per query block)
      f32x4 st[4][2];
#pragma unroll
      for (int sb = 0; sb < 4; ++sb) {
        bf16x8 kf[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          kf[c] = __builtin_bit_cast(bf16x8, kt[(sb * 16 + ln) * 16 + ((4 * c + lg) ^ ln)]);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < 4; ++c)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c], qf[qb][c], acc, 0, 0, 0);
          st[sb][qb] = acc;
        }
      }
      // Running softmax (base 2) per query block.  First the maxima of both blocks and the rare
      // rescaling (behind a wavefront-uniform branch), then exponentials and the second product in
      // one straight run of code, so that the MFMAs of one query block can be scheduled under the
      // exponentials of the other.
      if (key0 + kTK > n) {  // wavefront-uniform: the block sticks out of the sequence
#pragma unroll
        for (int sb = 0; sb < 4; ++sb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (key0 + sb * 16 + 4 * lg + e >= n) st[sb][0][e] = st[sb][1][e] = -INFINITY;
      }
      float m_use[2], m_new[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        float mx = -INFINITY;
#pragma unroll
        for (int sb = 0; sb < 4; ++sb)
#pragma unroll
          for (int e = 0; e < 4; ++e) mx = fmaxf(mx, st[sb][qb][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        // The reference point of the exponentials follows the running maximum lazily: it moves only
        // when the maximum has grown by more than kLazy (base-2 units) since it was last set, so
        // probabilities reach at most 2^kLazy (harmless in float32 sums and in a bf16 pair) and the
        // result is the same quotient.  With 32 queries per wavefront some maximum moves in most
        // blocks; by more than kLazy hardly ever after the first ones.
        const float mb = mx * sl2e;
        m_new[qb] = mb > m_run[qb] + kLazy ? mb : m_run[qb];
        m_use[qb] = m_new[qb] == -INFINITY ? 0.f : m_new[qb];
      }
      // the accumulators are rescaled only in the blocks in which some query's reference moved
      if (__builtin_amdgcn_ballot_w64(m_new[0] != m_run[0] || m_new[1] != m_run[1]) != 0) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          // 1 where nothing moved, 0 while nothing has been seen yet
          const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_use[qb]);
          l_run[qb] *= alpha;
          m_run[qb] = m_new[qb];
#pragma unroll
          for (int db = 0; db < 8; ++db) {
            o_acc[qb][db][0] *= alpha;
            o_acc[qb][db][1] *= alpha;
            o_acc[qb][db][2] *= alpha;
            o_acc[qb][db][3] *= alpha;
          }
        }
      }
      // Probabilities as a bf16 pair (high part + remainder: as single bf16 values they cost 11 % of
      // the step's distance from the float64 evaluation at full depth, more than the 2e-2 budget
      // has left), laid out as the B operand of the second product: MFMA k-slot 8*lg + t of half h is key
      // key0 + (2h + t/4)*16 + 4*lg + t%4.  (The hardware's 2^x as it is: the arguments are <= 0, and
      // results below the normal range, which it flushes to zero, are far below anything a bf16
      // probability can carry.)
      // The exponentials of the block's second 32 keys are dealt out between the MFMAs of its first
      // 32 (eight pieces of four probabilities, one per dim block).  That buys little here: on this
      // chip an MFMA with VALU instructions behind it takes its 16 cycles plus most of theirs
      // (measured: MFMA alone 16.9 cycles, with 4 v_fma 34.6, with 8 43.4 per MFMA at four
      // wavefronts per SIMD), so the block costs about the sum of its matrix and vector cycles and
      // what counts is the number of vector instructions per key.
      bf16x8 pf[2][2], pl[2][2];
      float psum[2] = {0.f, 0.f};
      auto exp_piece = [&](int qb, int sb, int e) {  // probabilities e, e+1 of sub-block sb
        const float e0 = __builtin_amdgcn_exp2f(fmaf(st[sb][qb][e], sl2e, -m_use[qb]));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(st[sb][qb][e + 1], sl2e, -m_use[qb]));
        psum[qb] += e0;
        psum[qb] += e1;
        const uint32_t hi = pack_bf16x2(e0, e1);
        reinterpret_cast<uint32_t*>(&pf[qb][sb / 2])[(sb % 2) * 2 + e / 2] = hi;
        reinterpret_cast<uint32_t*>(&pl[qb][sb / 2])[(sb % 2) * 2 + e / 2] =
            pack_bf16x2(e0 - __uint_as_float(hi << 16), e1 - __uint_as_float(hi & 0xffff0000u));
      };
      // O^T[dim][query] += V^T[dim][key] P^T[key][query] for dim block db and key half h
      auto pv_piece = [&](int db, int h) {
        typedef v4i16_t __attribute__((address_space(3))) * lds_v4;
        const v4i16_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vt + voff[db] + (2 * h) * 4096));
        const v4i16_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vt + voff[db] + (2 * h + 1) * 4096));
        typedef short v8i16_t __attribute__((ext_vector_type(8)));
        const v8i16_t both = {r0[0], r0[1], r0[2], r0[3], r1[0], r1[1], r1[2], r1[3]};
        const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          o_acc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qb][h], o_acc[qb][db], 0, 0, 0);
          o_acc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl[qb][h], o_acc[qb][db], 0, 0, 0);
        }
      };
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int e = 0; e < 4; e += 2) exp_piece(qb, sb, e);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        pv_piece(db, 0);
        exp_piece(db / 4, 2 + (db / 2) % 2, (db % 2) * 2);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int db = 0; db < 8; ++db) pv_piece(db, 1);
      l_run[0] += psum[0];
      l_run[1] += psum[1];
    }
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb)
    attn_finish(o_acc[qb], m_run[qb], l_run[qb], i0 + qb * 16 + ln, Mq, b, a, ks, KS, H_q, lg, out, part);
}

template <bool PAGED>
__global__ __launch_bounds__(256, 2) void k_attn_tile(const bf16_t* __restrict__ q, int Mq,
                                                      const bf16_t* __restrict__ kc,
                                                      const bf16_t* __restrict__ vc, int n, int H_q,
                                                      int H_kv, int KS, bf16_t* __restrict__ out,
                                                      float* __restrict__ part,
                                                      const int* __restrict__ rmap) {
  attn_tile_body<PAGED>(q, Mq, kc, vc, n, H_q, H_kv, KS, out, part, rmap);
}

// ---- few queries ---------------------------------------------------------------------
// k_attn_few<QB>: fewer than 128 queries per sequence (adaptive steps).  A workgroup is 16 * QB queries of one head
// against a range of keys; each of its four wavefronts walks every fourth 32-key block of the range
// by itself -- K and V tile from global memory straight into a two-stage ring in its own part of the
// LDS, no barrier anywhere in the walk -- and carries all the workgroup's queries, so that every fragment it
// reads feeds QB products.  The wavefronts' (O, m, l) meet in LDS.  V fragments come out of the
// row-major tile with transposing reads, as in k_attn_tile (32 keys here).
template <int QB, bool PAGED>
__device__ __forceinline__ void attn_few_body(const bf16_t* __restrict__ q, int Mq,
                                              const bf16_t* __restrict__ kc,
                                              const bf16_t* __restrict__ vc, int n, int H_q,
                                              int H_kv, int KS, bf16_t* __restrict__ out,
                                              float* __restrict__ part,
                                              const int* __restrict__ rmap) {
  constexpr int QT = 16 * QB;
  constexpr int kTile = 32 * 16;                  // 16-byte slots of a 32-key tile
  constexpr int kWaveVecs = 2 * 2 * kTile;        // [stage][K tile, V tile]
  constexpr int kOS = kDH + 4;                    // float32 row of the hand-over
  // Queries through LDS as well, a copy per wavefront (four do not fit): with them loaded into registers the
  // compiler waits for everything in flight, both blocks of the ring, in front of the first product.
  constexpr bool kQLds = QB <= 2;
  constexpr int kQVecs = kQLds ? QT * 16 : 0;
  constexpr int kRing = 4 * (kWaveVecs + kQVecs);
  constexpr int kHand = (4 * QT * kOS + 8 * QT) / 4;
  __shared__ __attribute__((aligned(1024))) uint4 smem[kRing > kHand ? kRing : kHand];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;  // scalar
  const int ln = lane % 16, lg = lane / 16;
  const AttnWork wk = attn_work_tile((Mq + QT - 1) / QT, H_q, H_kv, KS);
  const int a = wk.a, b = wk.b, ks = wk.ks;
  const int d_q = H_q * kDH, d_kv = H_kv * kDH;
  const int kv = a / (H_q / H_kv);
  const int i0 = wk.qtile * QT;
  const bf16_t* K = kc + kv * kDH;
  const bf16_t* V = vc + kv * kDH;
  const int seq0 = b * n;
  uint4* ring = smem + wave * (kWaveVecs + kQVecs);

  const int nblk = (n + 31) / 32;
  const int per = (nblk + KS - 1) / KS;
  const int blk0 = ks * per;
  const int blk1 = min(nblk, blk0 + per);
  const int nb = (blk1 - blk0 - wave + 3) / 4;    // blocks blk0 + wave, + 4, ... of this wavefront

  // loader: a tile is 8 instructions of 4 keys x 256 bytes; lane l: key 4j + l/16, slot l%16, chunk
  // slot ^ (key % 16)
  int chunk[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) chunk[j] = ((lane % 16) ^ (4 * j + lane / 16)) * 8;
  // block i of this wavefront; blocks past its last one repeat that (never used: the number of loads in
  // flight stays the same in every iteration)
  auto key0_of = [&](int i) { return (blk0 + wave + 4 * min(i, nb - 1)) * 32; };
  auto rows_of = [&](int i, int (&cr)[8]) {
    const int key0 = key0_of(i);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int kr = seq0 + min(key0 + 4 * j + lane / 16, n - 1);  // keys past the end are masked in the scores
      cr[j] = PAGED ? rmap[kr] : kr;
    }
  };
  auto issue = [&](const bf16_t* T, const int (&cr)[8], uint4* tile) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      __builtin_amdgcn_global_load_lds(T + static_cast<size_t>(cr[j]) * d_kv + chunk[j % 4], tile + j * 64, 16, 0, 0);
  };

  // Q fragments: lane (query ln, group lg) holds dims 32c + 8lg .. +8 (padded queries compute a duplicate
  // that is never stored)
  bf16x8 qf[QB][4];
  uint4* qtile = ring + kWaveVecs;
  if (kQLds) {
#pragma unroll
    for (int j = 0; j < 4 * QB; ++j) {
      const int qi = min(i0 + 4 * j + lane / 16, Mq - 1);
      __builtin_amdgcn_global_load_lds(q + (static_cast<size_t>(b) * Mq + qi) * d_q + a * kDH + chunk[j % 4],
                                       qtile + j * 64, 16, 0, 0);
    }
  } else {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int qi = min(i0 + qb * 16 + ln, Mq - 1);
      const bf16_t* qr = q + (static_cast<size_t>(b) * Mq + qi) * d_q + a * kDH + lg * 8;
#pragma unroll
      for (int c = 0; c < 4; ++c) qf[qb][c] = *reinterpret_cast<const bf16x8*>(qr + c * 32);
    }
  }
  const float sl2e = 1.4426950408889634f / sqrtf(static_cast<float>(kDH));  // scale * log2(e)
  float m_run[QB], l_run[QB];
  f32x4 o_acc[QB][8];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.f;
#pragma unroll
    for (int db = 0; db < 8; ++db) o_acc[qb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // transposing reads (see k_attn_tile): byte offset inside a V tile for dim block db, sub-block 0
  const int krow = 4 * lg + ln / 4;
  int voff[8];
#pragma unroll
  for (int db = 0; db < 8; ++db)
    voff[db] = (krow * 16 + ((2 * db + (ln % 4) / 2) ^ krow)) * 16 + (ln % 2) * 8;

  if (nb > 0) {
    int cr[8];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      rows_of(s, cr);
      issue(K, cr, ring + s * 2 * kTile);
      issue(V, cr, ring + s * 2 * kTile + kTile);
    }
    rows_of(2, cr);
    // (paged layout: nothing keeps the row-map lookups behind the tile loads in front of them; counts that hold
    // wherever the compiler has put them)
    if (kQLds) {
      wait_vmcnt<32>();  // the queries: older than the 32 tile loads
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          qf[qb][c] = __builtin_bit_cast(bf16x8, qtile[(qb * 16 + ln) * 16 + ((4 * c + lg) ^ ln)]);
    }
    if (PAGED) wait_vmcnt<16>();  // block 0: older than the 16 loads of block 1
    for (int i = 0; i < nb; ++i) {
      // block i has landed: block i + 1 (16 loads), and in the paged layout the lookups of the iteration
      // before (8, on either side of those loads), may be in flight
      wait_vmcnt<16 + (PAGED ? 8 : 0)>();
      __builtin_amdgcn_sched_barrier(0);
      uint4* kt = ring + (i & 1) * 2 * kTile;
      const char* vt = reinterpret_cast<const char*>(kt + kTile);
      const int key0 = (blk0 + wave + 4 * i) * 32;
      f32x4 st[2][QB];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        bf16x8 kf[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          kf[c] = __builtin_bit_cast(bf16x8, kt[(sb * 16 + ln) * 16 + ((4 * c + lg) ^ ln)]);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < 4; ++c)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c], qf[qb][c], acc, 0, 0, 0);
          st[sb][qb] = acc;
        }
      }
      if (key0 + 32 > n) {  // wavefront-uniform: the block sticks out of the sequence
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (key0 + sb * 16 + 4 * lg + e >= n) {
#pragma unroll
              for (int qb = 0; qb < QB; ++qb) st[sb][qb][e] = -INFINITY;
            }
      }
      // running softmax (base 2); the reference point follows the maximum lazily (see k_attn_tile)
      float m_use[QB], m_new[QB];
      bool moved = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float mx = -INFINITY;
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int e = 0; e < 4; ++e) mx = fmaxf(mx, st[sb][qb][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mb = mx * sl2e;
        m_new[qb] = mb > m_run[qb] + kLazy ? mb : m_run[qb];
        m_use[qb] = m_new[qb] == -INFINITY ? 0.f : m_new[qb];
        moved |= m_new[qb] != m_run[qb];
      }
      if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_use[qb]);
          l_run[qb] *= alpha;
          m_run[qb] = m_new[qb];
#pragma unroll
          for (int db = 0; db < 8; ++db) o_acc[qb][db] *= alpha;
        }
      }
      // probabilities as a bf16 pair (high part + remainder), in the second product's operand layout
      bf16x8 pf[QB], pl[QB];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(st[sb][qb][e], sl2e, -m_use[qb]));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(st[sb][qb][e + 1], sl2e, -m_use[qb]));
            l_run[qb] += e0;
            l_run[qb] += e1;
            const uint32_t hi = pack_bf16x2(e0, e1);
            reinterpret_cast<uint32_t*>(&pf[qb])[sb * 2 + e / 2] = hi;
            reinterpret_cast<uint32_t*>(&pl[qb])[sb * 2 + e / 2] =
                pack_bf16x2(e0 - __uint_as_float(hi << 16), e1 - __uint_as_float(hi & 0xffff0000u));
          }
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        typedef v4i16_t __attribute__((address_space(3))) * lds_v4;
        typedef short v8i16_t __attribute__((ext_vector_type(8)));
        const v4i16_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vt + voff[db]));
        const v4i16_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(vt + voff[db] + 4096));
        const v8i16_t both = {r0[0], r0[1], r0[2], r0[3], r1[0], r1[1], r1[2], r1[3]};
        const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          o_acc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qb], o_acc[qb][db], 0, 0, 0);
          o_acc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl[qb], o_acc[qb][db], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // This wavefront's reads of the stage are complete: block i + 2 takes it.  (Paged layout: with tile loads in
      // flight the compiler waits for a lookup with vmcnt(0), so here block i + 1 lands first and a wavefront has one
      // block in flight, not two.  The lookups of the block after go out last: not one of them is waited for fresh.)
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      issue(K, cr, kt);
      issue(V, cr, kt + kTile);
      rows_of(i + 3, cr);
    }
  }
  wait_vmcnt<0>();  // the repeated loads past the range, before the ring is overwritten
  __syncthreads();
  float* hand = reinterpret_cast<float*>(smem);                 // [wavefront][query][kOS]
  float* ml = hand + 4 * QT * kOS;                              // [wavefront][query] m, then l
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    l_run[qb] += __shfl_xor(l_run[qb], 16, 64);
    l_run[qb] += __shfl_xor(l_run[qb], 32, 64);
#pragma unroll
    for (int db = 0; db < 8; ++db)
      *reinterpret_cast<f32x4*>(&hand[(wave * QT + qb * 16 + ln) * kOS + db * 16 + 4 * lg]) = o_acc[qb][db];
    if (lg == 0) {
      ml[wave * QT + qb * 16 + ln] = m_run[qb];
      ml[4 * QT + wave * QT + qb * 16 + ln] = l_run[qb];
    }
  }
  __syncthreads();
  // 16 threads per query, eight dims each; the wavefronts' parts in order
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int ql = qb * 16 + threadIdx.x / 16, t8 = (threadIdx.x % 16) * 8;
    const int iq = i0 + ql;
    if (iq >= Mq) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, ml[w * QT + ql]);
    float L = 0.f, o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float mw = ml[w * QT + ql];
      const float f = mw == -INFINITY ? 0.f : exp2f(mw - M);
      L += ml[4 * QT + w * QT + ql] * f;
      const float* ow = &hand[(w * QT + ql) * kOS + t8];
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(ow), x1 = *reinterpret_cast<const f32x4*>(ow + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] += x0[e] * f;
        o[4 + e] += x1[e] * f;
      }
    }
    if (KS == 1) {
      const float inv = 1.0f / L;
      // (two 8-byte stores, as the other kernels: a result need not start at 16 bytes)
      uint2* dst = reinterpret_cast<uint2*>(out + (static_cast<size_t>(b) * Mq + iq) * d_q + a * kDH + t8);
      dst[0] = make_uint2(pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv));
      dst[1] = make_uint2(pack_bf16x2(o[4] * inv, o[5] * inv), pack_bf16x2(o[6] * inv, o[7] * inv));
    } else {
      float* w = part + ((static_cast<size_t>(b) * Mq + iq) * H_q + a) * KS * (kDH + 2) +
                 static_cast<size_t>(ks) * (kDH + 2);
#pragma unroll
      for (int e = 0; e < 8; e += 2) *reinterpret_cast<float2*>(w + t8 + e) = make_float2(o[e], o[e + 1]);
      if (t8 == 0) {
        w[kDH] = M;
        w[kDH + 1] = L;
      }
    }
  }
}

template <int QB, bool PAGED>
__global__ __launch_bounds__(256, QB <= 2 ? 2 : 1) void k_attn_few(const bf16_t* __restrict__ q, int Mq,
                                                     const bf16_t* __restrict__ kc,
                                                     const bf16_t* __restrict__ vc, int n, int H_q,
                                                     int H_kv, int KS, bf16_t* __restrict__ out,
                                                     float* __restrict__ part,
                                                     const int* __restrict__ rmap) {
  attn_few_body<QB, PAGED>(q, Mq, kc, vc, n, H_q, H_kv, KS, out, part, rmap);
}

// out[query][head][:] = sum_r O_r 2^(m_r - M) / sum_r l_r 2^(m_r - M), in key-range order.
// One wavefront per (query, head), two dims per lane.
template <int SLOTS>
__global__ __launch_bounds__(64) void k_attn_merge(const float* __restrict__ part, int KS,
                                                   bf16_t* __restrict__ out) {
  const size_t qh = static_cast<size_t>(blockIdx.x);  // (b*Mq + iq)*H_q + a
  const float* w = part + qh * KS * (kDH + 2);
  // All SLOTS >= KS slots are loaded before the first use (slots past KS re-read the last
  // valid one and get weight zero): a loop over the runtime count would wait for each load.
  const int dim = threadIdx.x * 2;
  float mr[SLOTS], lr[SLOTS];
  float2 o[SLOTS];
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    const float* wr = w + min(r, KS - 1) * (kDH + 2);
    mr[r] = wr[kDH];
    lr[r] = wr[kDH + 1];
    o[r] = *reinterpret_cast<const float2*>(wr + dim);
  }
  float M = -INFINITY;
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) M = fmaxf(M, mr[r]);
  float L = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    const float f = (r >= KS || mr[r] == -INFINITY) ? 0.f : exp2f(mr[r] - M);
    L += lr[r] * f;
    o0 += o[r].x * f;
    o1 += o[r].y * f;
  }
  const uint32_t t = static_cast<uint32_t>(f32_to_bf16(o0 / L)) |
                     (static_cast<uint32_t>(f32_to_bf16(o1 / L)) << 16);
  *reinterpret_cast<uint32_t*>(out + qh * kDH + dim) = t;
}

}  // namespace

// Keys are split only while (workgroups without split) * KS stays within 256 (k_attn_tile: 128 queries per
// workgroup; the others 64 or fewer), so this bounds the partial results.
size_t attention_scratch_floats() { return static_cast<size_t>(kQT) * 1024 * (kDH + 2); }

bool attention_supported(int dtype, int d_h, int n) {
  if (dtype == 1 && d_h == kDH) return true;
  return static_cast<size_t>(d_h + n) * sizeof(float) <= 60 * 1024;
}

// Fewer than 128 queries per sequence: three kernels, by estimated time in us, fitted to 3336 shapes (1 to 16 sequences, 1
// to 127 queries, 50 to 4608 keys, heads 32, 28/4, 7/1 and 8) that were timed with every kernel and number of key
// ranges, on keys and values that mostly no cache holds.  MB: keys and values; P: MB of partial results, written and read.
//   few<QB>, KS ranges   1.4 + rounds of 256 workgroups (one per CU) x (2.8 / 3.85 / 7.0 + 1.07 / 1.37 / 2.08 per 32-key block
//                        of a wavefront's walk, at QB = 1 / 2 / 4) + MB / 14, and 2.1 + P / 4.3 for a merge launch
//   walk, whole ranges   4.5 + 1.0 per block + MB / 14 for up to 256 workgroups (64 queries each, four wavefronts on the
//                        same block), 1.4 per block for 512, which share the CUs; again for every further 512
//   mfma                 8.0 + P / 5 with its merge launch: ranges of three blocks, everything fetched at once; only while
//                        they do not share CUs
// The choice is on average 0.7 % slower than the best of all (at worst 30 %: 10 us), and nowhere more than 5 % slower than
// mfma and walk alone with up to 512 workgroups, which were 36 % slower on average.  (A first estimate counted no fixed
// time per round of k_attn_few and gave it launches of several rounds that belong to walk: 16 sequences, 100 queries, 100
// keys, 28/4 heads 41.5 us, now 21.5; 8, 51, 300, 32 22.2 -> 17.2; 2, 20, 2500, 32 24.3 -> 22.)
FewPlan plan_attention_few(int B, int Mq, int n, int H_q, int H_kv, bool split_keys) {
  const int nblk = (n + 31) / 32;
  const double t_kv = 4.0 * B * n * H_kv * kDH / 1e6 / 14.0;
  const double mb_part = static_cast<double>(B) * Mq * H_q * (kDH + 2) * 8.0 / 1e6;  // per key range
  const int base = B * ((Mq + kQT - 1) / kQT) * H_q, rem = base % 512;
  FewPlan best{0, 1};  // walk
  double t_best = base / 512 * (4.5 + 1.4 * nblk) + t_kv;
  if (rem > 0) t_best += 4.5 + nblk * (rem <= 256 ? 1.0 : 1.4);
  double margin = 0.97;  // (walk is taken at a tie: its estimate strays less)
  for (int qb = 1; qb <= 4; qb *= 2) {
    const int tiles = B * ((Mq + 16 * qb - 1) / (16 * qb)) * H_q;
    const double start = qb == 1 ? 2.8 : qb == 2 ? 3.85 : 7.0, block = qb == 1 ? 1.07 : qb == 2 ? 1.37 : 2.08;
    for (int s = 1; s <= kMaxKeySplit; s *= 2) {
      if (s > 1 && (!split_keys || tiles * s > 256 || 2 * s > nblk)) break;
      const int blocks = ((nblk + s - 1) / s + 3) / 4;
      double t = 1.4 + (tiles * s + 255) / 256 * (start + blocks * block) + t_kv;
      if (s > 1) t += 2.1 + s * mb_part / 4.3;
      if (t < t_best * margin) { t_best = t; best = FewPlan{qb, s}; margin = 0.98; }
    }
  }
  const int ks3 = (nblk + kPreload - 1) / kPreload;
  if (split_keys && ks3 >= 2 && ks3 <= kMaxKeySplit && base * ks3 <= 256 && 8.0 + ks3 * mb_part / 5.0 < t_best)
    best = FewPlan{-1, ks3};
  return best;
}

void launch_attention(int dtype, const void* q, int B, int Mq, const void* k_cache,
                      const void* v_cache, int n, int H_q, int H_kv, int d_h, void* out,
                      float* scratch, hipStream_t st, const int* rmap) {
  if (B <= 0 || Mq <= 0 || n <= 0) return;
  if (dtype == 1 && d_h == kDH) {
    const bf16_t* qq = static_cast<const bf16_t*>(q);
    const bf16_t* kk = static_cast<const bf16_t*>(k_cache);
    const bf16_t* vv = static_cast<const bf16_t*>(v_cache);
    bf16_t* oo = static_cast<bf16_t*>(out);
    if (Mq >= kTQ) {
      // many queries per (sequence, head): 128-query tiles; the keys are split only when the
      // queries alone would leave at least half of the CUs without a workgroup
      const int base128 = B * ((Mq + kTQ - 1) / kTQ) * H_q;
      const int nblk64 = (n + kTK - 1) / kTK;
      int KS = 1;
      if (scratch != nullptr && 2 * base128 <= 256) {
        KS = 256 / base128;
        if (KS > 8) KS = 8;
        if (KS > nblk64 / 2) KS = nblk64 / 2 > 0 ? nblk64 / 2 : 1;
      }
      const dim3 grid(base128 * KS);
      if (rmap)
        hipLaunchKernelGGL(k_attn_tile<true>, grid, dim3(256), 0, st, qq, Mq, kk, vv, n, H_q, H_kv, KS, oo,
                           scratch, rmap);
      else
        hipLaunchKernelGGL(k_attn_tile<false>, grid, dim3(256), 0, st, qq, Mq, kk, vv, n, H_q, H_kv, KS, oo,
                           scratch, rmap);
      if (KS > 1)
        hipLaunchKernelGGL(k_attn_merge<8>, dim3(B * Mq * H_q), dim3(64), 0, st, scratch, KS, oo);
      return;
    }
    const FewPlan pl = plan_attention_few(B, Mq, n, H_q, H_kv, scratch != nullptr);
    const int KS = pl.KS, base = B * ((Mq + kQT - 1) / kQT) * H_q;
#define DLLMC_ATTN(KERNEL, GRID) \
  hipLaunchKernelGGL(KERNEL, dim3(GRID), dim3(256), 0, st, qq, Mq, kk, vv, n, H_q, H_kv, KS, oo, scratch, rmap)
#define DLLMC_ATTN_WALK(KERNEL) \
  hipLaunchKernelGGL(KERNEL, dim3(base), dim3(256), 0, st, qq, Mq, kk, vv, n, H_q, H_kv, oo, rmap)
#define DLLMC_ATTN_FEW(Q)                                                                        \
  do {                                                                                           \
    const int grid_ = B * ((Mq + 16 * Q - 1) / (16 * Q)) * H_q * KS;                              \
    if (rmap) DLLMC_ATTN((k_attn_few<Q, true>), grid_); else DLLMC_ATTN((k_attn_few<Q, false>), grid_); \
  } while (0)
    switch (pl.QB) {
      case -1: if (rmap) DLLMC_ATTN(k_attn_mfma<true>, base * KS); else DLLMC_ATTN(k_attn_mfma<false>, base * KS); break;
      case 0: if (rmap) DLLMC_ATTN_WALK(k_attn_walk<true>); else DLLMC_ATTN_WALK(k_attn_walk<false>); break;
      case 1: DLLMC_ATTN_FEW(1); break;
      case 2: DLLMC_ATTN_FEW(2); break;
      default: DLLMC_ATTN_FEW(4); break;
    }
#undef DLLMC_ATTN_FEW
#undef DLLMC_ATTN_WALK
#undef DLLMC_ATTN
    if (KS > 8)
      hipLaunchKernelGGL(k_attn_merge<kMaxKeySplit>, dim3(B * Mq * H_q), dim3(64), 0, st, scratch, KS,
                         oo);
    else if (KS > 1)
      hipLaunchKernelGGL(k_attn_merge<8>, dim3(B * Mq * H_q), dim3(64), 0, st, scratch, KS, oo);
    return;
  }
  // float32 arithmetic on the matrix cores: operands in whole aligned 16-byte (bf16: 8-byte) pieces
  const uintptr_t low = reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_cache) |
                        reinterpret_cast<uintptr_t>(v_cache);
  if ((d_h == 64 || (d_h == kDH && dtype == 0)) && low % (dtype == 1 ? 8 : 16) == 0) {
    const dim3 grid((Mq + 15) / 16, H_q, B);
#define DLLMC_ATTN(T, D, PG)                                                                           \
  hipLaunchKernelGGL((k_attn_f32<T, D, PG>), grid, dim3(64 * kFW), 0, st, static_cast<const T*>(q), Mq, \
                     static_cast<const T*>(k_cache), static_cast<const T*>(v_cache), n, H_q, H_kv,      \
                     static_cast<T*>(out), rmap)
    if (dtype == 1 && rmap) DLLMC_ATTN(bf16_t, 64, true);
    else if (dtype == 1) DLLMC_ATTN(bf16_t, 64, false);
    else if (d_h == 64 && rmap) DLLMC_ATTN(float, 64, true);
    else if (d_h == 64) DLLMC_ATTN(float, 64, false);
    else if (rmap) DLLMC_ATTN(float, 128, true);
    else DLLMC_ATTN(float, 128, false);
#undef DLLMC_ATTN
    return;
  }
  const size_t lds = static_cast<size_t>(d_h + n) * sizeof(float);
  if (dtype == 1)
    hipLaunchKernelGGL(k_attn_simple<bf16_t>, dim3(Mq, H_q, B), dim3(64), lds, st,
                       static_cast<const bf16_t*>(q), Mq, static_cast<const bf16_t*>(k_cache),
                       static_cast<const bf16_t*>(v_cache), n, H_q, H_kv, d_h,
                       static_cast<bf16_t*>(out), rmap);
  else
    hipLaunchKernelGGL(k_attn_simple<float>, dim3(Mq, H_q, B), dim3(64), lds, st,
                       static_cast<const float*>(q), Mq, static_cast<const float*>(k_cache),
                       static_cast<const float*>(v_cache), n, H_q, H_kv, d_h,
                       static_cast<float*>(out), rmap);
}

}  // namespace dllmc
