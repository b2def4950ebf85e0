// Kernels of the closed denoising loop around the cached step (paper Sec. 3.1: greedy estimate
// of the clean sequence, transition to the next state by low-confidence remasking):
//   k_embed_gather    token ids -> embedded rows
//   k_elig_scores     which response positions are still masked inside the current block
//   k_final_norm      RMSNorm with the final gain of the listed rows, compact output
//   k_head_partial    per row and run of logits: maximum, sum of exponentials, first index of the
//                     maximum; k_head_merge: the row's greedy token (lowest id among equal logits) and its
//                     softmax probability from those, or from the ones that the vocabulary projection of
//                     up to 640 rows leaves instead of logits (k_gemm_mid_head)
//   k_apply_tokens    the chosen positions take their greedy token
// The vocabulary projection itself is a gathered linear map (kernels_gemm.hip); the choice of
// the positions is the integer-exact bottom-k selection (kernels_select.hip) on the negated
// confidences.
#include <cmath>

#include "common.hpp"

namespace dllmc {

namespace {

constexpr int kThreads = 256;
constexpr int kNW = kThreads / kWave;

template <typename T>
__global__ __launch_bounds__(kThreads) void k_embed_gather(const T* __restrict__ table,
                                                           const int* __restrict__ tokens, int d,
                                                           int vocab_rows, T* __restrict__ out) {
  const int row = blockIdx.x;
  int tok = tokens[row];
  tok = tok < 0 ? 0 : (tok >= vocab_rows ? vocab_rows - 1 : tok);  // never read outside the table
  const T* src = table + static_cast<size_t>(tok) * d;
  T* dst = out + static_cast<size_t>(row) * d;
  constexpr int V = 16 / sizeof(T);  // elements per 16-byte vector
  if (d % V == 0) {
    const uint4* s4 = reinterpret_cast<const uint4*>(src);
    uint4* d4 = reinterpret_cast<uint4*>(dst);
    for (int c = threadIdx.x; c < d / V; c += kThreads) d4[c] = s4[c];
  } else {
    for (int c = threadIdx.x; c < d; c += kThreads) dst[c] = src[c];
  }
}

// elig[b][j] = 0 if response position j of sequence b holds mask_id and lo <= j < hi, else 1;
// neg_conf[b][j] = +inf and x0[b][j] = -1 (overwritten for the eligible positions later).
__global__ __launch_bounds__(kThreads) void k_elig_scores(const int* __restrict__ tokens, int B,
                                                          int n, int L_p, int lo, int hi,
                                                          int mask_id, float* __restrict__ elig,
                                                          float* __restrict__ neg_conf,
                                                          int* __restrict__ x0) {
  const int L_r = n - L_p;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= B * L_r) return;
  const int b = i / L_r, j = i % L_r;
  const bool e = j >= lo && j < hi && tokens[b * n + L_p + j] == mask_id;
  elig[i] = e ? 0.0f : 1.0f;
  neg_conf[i] = INFINITY;
  x0[i] = -1;
}

// eight (bf16) or four (float32) neighbouring elements of a row, as one 16-byte access
template <typename T> struct Piece {
  static constexpr int N = 16 / sizeof(T);
  float v[N];
  __device__ __forceinline__ void load(const T* p) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < N; ++i)
      v[i] = sizeof(T) == 4 ? __uint_as_float(w[i % 4])
                            : __uint_as_float(i % 2 ? w[i / 2 % 4] & 0xffff0000u : w[i / 2 % 4] << 16);
  }
  __device__ __forceinline__ void store(T* p) const {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = sizeof(T) == 4 ? __float_as_uint(v[i % N])
                            : static_cast<uint32_t>(f32_to_bf16(v[2 * i % N])) |
                                  (static_cast<uint32_t>(f32_to_bf16(v[(2 * i + 1) % N])) << 16);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
  }
};

// VEC: rows in whole aligned 16-byte pieces.  A row of up to two pieces per thread (bf16: 4096 wide) stays in
// registers, with the gain's pieces requested under the reduction: one trip to memory (with 2-byte accesses
// and the row read twice 10 us for 100 rows of 4096, now 5).
template <typename T, bool VEC>
__global__ __launch_bounds__(kThreads) void k_final_norm(const T* __restrict__ hidden,
                                                         const int* __restrict__ rows, int d,
                                                         float eps, const T* __restrict__ gain,
                                                         T* __restrict__ z) {
  __shared__ float red[kNW];
  constexpr int N = Piece<T>::N, KEEP = 2;
  const int i = blockIdx.x;
  const int row = rows ? rows[i] : i;
  const T* src = hidden + static_cast<size_t>(row) * d;
  T* dst = z + static_cast<size_t>(i) * d;
  float ss = 0.f;
  if (VEC) {
    Piece<T> x[KEEP], g[KEEP];
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
      const int c = min((k * kThreads + static_cast<int>(threadIdx.x)) * N, d - N);
      x[k].load(src + c);
      g[k].load(gain + c);
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
      if ((k * kThreads + static_cast<int>(threadIdx.x)) * N < d) {
#pragma unroll
        for (int e = 0; e < N; ++e) ss += x[k].v[e] * x[k].v[e];
      }
    for (int c = (KEEP * kThreads + static_cast<int>(threadIdx.x)) * N; c < d; c += kThreads * N) {
      Piece<T> y;
      y.load(src + c);
#pragma unroll
      for (int e = 0; e < N; ++e) ss += y.v[e] * y.v[e];
    }
    ss = block_sum<kNW>(ss, red);
    const float rstd = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
      const int c = (k * kThreads + static_cast<int>(threadIdx.x)) * N;
      if (c < d) {
#pragma unroll
        for (int e = 0; e < N; ++e) x[k].v[e] = x[k].v[e] * rstd * g[k].v[e];
        x[k].store(dst + c);
      }
    }
    for (int c = (KEEP * kThreads + static_cast<int>(threadIdx.x)) * N; c < d; c += kThreads * N) {
      Piece<T> y, gy;
      y.load(src + c);
      gy.load(gain + c);
#pragma unroll
      for (int e = 0; e < N; ++e) y.v[e] = y.v[e] * rstd * gy.v[e];
      y.store(dst + c);
    }
    return;
  }
  for (int c = threadIdx.x; c < d; c += kThreads) {
    const float v = ldf(src + c);
    ss += v * v;
  }
  ss = block_sum<kNW>(ss, red);
  const float rstd = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
  for (int c = threadIdx.x; c < d; c += kThreads) stf(dst + c, ldf(src + c) * rstd * ldf(gain + c));
}

// running (maximum, sum of exp(l - maximum), index of the first maximum)
__device__ __forceinline__ HeadPart soft_merge(const HeadPart& p, const HeadPart& q) {
  HeadPart r;
  r.m = fmaxf(p.m, q.m);
  // (nothing but -inf so far: the sum is 0, or NaN)
  r.s = (p.m == -INFINITY ? p.s : p.s * expf(p.m - r.m)) + (q.m == -INFINITY ? q.s : q.s * expf(q.m - r.m));
  r.a = p.m > q.m ? p.a : (q.m > p.m ? q.a : min(p.a, q.a));
  r.unused = 0;
  return r;
}

// the workgroup's partial results, lanes and then wavefronts in a fixed order; the total in thread 0
__device__ __forceinline__ HeadPart soft_reduce(HeadPart t, HeadPart* lds) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    HeadPart q;
    q.m = __shfl_xor(t.m, o, kWave);
    q.s = __shfl_xor(t.s, o, kWave);
    q.a = __shfl_xor(t.a, o, kWave);
    t = soft_merge(t, q);
  }
  if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    t = lds[0];
#pragma unroll
    for (int w = 1; w < kNW; ++w) t = soft_merge(t, lds[w]);
  }
  return t;
}

// Greedy token and confidence of row i: to x0[b][j] and conf[b][j] with rows (rows[i] = b*n + L_p + j),
// otherwise to x0[i] and conf[i]; conf = sign * probability.
__device__ __forceinline__ void head_store(const HeadPart& r, int i, const int* __restrict__ rows, int n,
                                           int L_p, float sign, int* __restrict__ x0,
                                           float* __restrict__ conf) {
  int o = i;
  if (rows) {
    const int row = rows[i];
    o = (row / n) * (n - L_p) + (row % n - L_p);
  }
  x0[o] = r.a;
  conf[o] = sign / r.s;
}

// Row blockIdx.x of the logits, columns of run blockIdx.y: one partial result per run, or (a single run) the
// row's token and confidence.  A thread takes 16 logits at a time: their maximum, then their
// exponentials against it (one per logit; merging them one by one into the running result took two and a
// chain of dependent instructions per logit: 92 us for 100 rows of 126464, one workgroup each).
template <bool VEC>
__global__ __launch_bounds__(kThreads) void k_head_partial(const float* __restrict__ logits, int vocab,
                                                           int run, HeadPart* __restrict__ part,
                                                           const int* __restrict__ rows, int n, int L_p,
                                                           float sign, int* __restrict__ x0,
                                                           float* __restrict__ conf) {
  __shared__ HeadPart lds[kNW];
  const int i = blockIdx.x;
  const float* l = logits + static_cast<size_t>(i) * vocab;
  const int c0 = blockIdx.y * run, c1 = min(vocab, c0 + run);
  HeadPart t{-INFINITY, 0.f, 0x7fffffff, 0};
  constexpr int W = VEC ? 4 : 1, U = 16 / W;  // U loads of W neighbouring logits
  for (int base = c0; base < c1; base += kThreads * 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = base + (u * kThreads + static_cast<int>(threadIdx.x)) * W;
      if (VEC) {
        const float4 f = *reinterpret_cast<const float4*>(l + min(c, vocab - 4));
        v[u * W] = f.x; v[u * W + 1 % W] = f.y; v[u * W + 2 % W] = f.z; v[u * W + 3 % W] = f.w;
      } else {
        v[u] = l[min(c, vocab - 1)];
      }
    }
    HeadPart q{-INFINITY, 0.f, 0x7fffffff, 0};
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int c = base + ((u / W) * kThreads + static_cast<int>(threadIdx.x)) * W + u % W;
      if (c < c1) q.m = fmaxf(q.m, v[u]);
    }
    const float mu = q.m == -INFINITY ? 0.f : q.m;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int c = base + ((u / W) * kThreads + static_cast<int>(threadIdx.x)) * W + u % W;
      if (c < c1) {
        q.s += expf(v[u] - mu);
        if (!(v[u] < q.m)) q.a = min(q.a, c);  // (a NaN, the only one past the maximum, counts as found)
      }
    }
    t = soft_merge(t, q);
  }
  t = soft_reduce(t, lds);
  if (threadIdx.x == 0) {
    if (part) part[static_cast<size_t>(i) * gridDim.y + blockIdx.y] = t;
    else head_store(t, i, rows, n, L_p, sign, x0, conf);
  }
}

// row blockIdx.x's n_part partial results -> token and confidence
__global__ __launch_bounds__(kThreads) void k_head_merge(const HeadPart* __restrict__ part, int n_part,
                                                         const int* __restrict__ rows, int n, int L_p,
                                                         float sign, int* __restrict__ x0,
                                                         float* __restrict__ conf) {
  __shared__ HeadPart lds[kNW];
  const int i = blockIdx.x;
  const HeadPart* p = part + static_cast<size_t>(i) * n_part;
  HeadPart t{-INFINITY, 0.f, 0x7fffffff, 0};
  for (int c0 = threadIdx.x; c0 < n_part; c0 += 4 * kThreads) {
    HeadPart q[4];  // four in flight
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = p[min(c0 + u * kThreads, n_part - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (c0 + u * kThreads < n_part) t = soft_merge(t, q[u]);
  }
  t = soft_reduce(t, lds);
  if (threadIdx.x == 0) head_store(t, i, rows, n, L_p, sign, x0, conf);
}

// tokens[b][L_p + chosen[b][t]] = x0[b][chosen[b][t]] for t < n_unmask
__global__ __launch_bounds__(kThreads) void k_apply_tokens(int* __restrict__ tokens, int B, int n,
                                                           int L_p, const int* __restrict__ chosen,
                                                           int chosen_stride, int n_unmask,
                                                           const int* __restrict__ x0) {
  const int L_r = n - L_p;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= B * n_unmask) return;
  const int b = i / n_unmask, t = i % n_unmask;
  const int j = chosen[b * chosen_stride + t];
  tokens[b * n + L_p + j] = x0[b * L_r + j];
}

__global__ __launch_bounds__(kThreads) void k_negate_f32(float* __restrict__ p, size_t count) {
  const size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i < count) p[i] = -p[i];
}

}  // namespace

void launch_negate_f32(float* p, size_t count, hipStream_t st) {
  if (count == 0) return;
  hipLaunchKernelGGL(k_negate_f32, dim3(static_cast<unsigned>((count + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, st, p, count);
}

void launch_embed_gather(int dtype, const void* table, int vocab_rows, const int* tokens, int rows,
                         int d, void* out, hipStream_t st) {
  if (rows <= 0) return;
  if (dtype == 1)
    hipLaunchKernelGGL(k_embed_gather<bf16_t>, dim3(rows), dim3(kThreads), 0, st,
                       static_cast<const bf16_t*>(table), tokens, d, vocab_rows,
                       static_cast<bf16_t*>(out));
  else
    hipLaunchKernelGGL(k_embed_gather<float>, dim3(rows), dim3(kThreads), 0, st,
                       static_cast<const float*>(table), tokens, d, vocab_rows,
                       static_cast<float*>(out));
}

void launch_elig_scores(const int* tokens, int B, int n, int L_p, int lo, int hi, int mask_id,
                        float* elig, float* neg_conf, int* x0, hipStream_t st) {
  const int total = B * (n - L_p);
  if (total <= 0) return;
  hipLaunchKernelGGL(k_elig_scores, dim3((total + kThreads - 1) / kThreads), dim3(kThreads), 0, st,
                     tokens, B, n, L_p, lo, hi, mask_id, elig, neg_conf, x0);
}

void launch_final_norm(int dtype, const void* hidden, const int* rows, int M, int d, float eps,
                       const void* gain, void* z, hipStream_t st) {
  if (M <= 0) return;
  const uintptr_t low = reinterpret_cast<uintptr_t>(hidden) | reinterpret_cast<uintptr_t>(gain) |
                        reinterpret_cast<uintptr_t>(z);
  const bool vec = low % 16 == 0 && d % (dtype == 1 ? 8 : 4) == 0;
#define DLLMC_FN(T, VEC)                                                                              \
  hipLaunchKernelGGL((k_final_norm<T, VEC>), dim3(M), dim3(kThreads), 0, st, static_cast<const T*>(hidden), \
                     rows, d, eps, static_cast<const T*>(gain), static_cast<T*>(z))
  if (dtype == 1 && vec) DLLMC_FN(bf16_t, true);
  else if (dtype == 1) DLLMC_FN(bf16_t, false);
  else if (vec) DLLMC_FN(float, true);
  else DLLMC_FN(float, false);
#undef DLLMC_FN
}

void launch_head_finalize(const float* logits, int M, int vocab, float* part, size_t part_floats,
                          const int* rows, int n, int L_p, float sign, int* x0, float* conf,
                          hipStream_t st) {
  if (M <= 0) return;
  // Runs of 4096 logits (one round of a workgroup), fewer and longer ones where the scratch is short of
  // room for their results, one if there is none.
  int runs = (vocab + 4095) / 4096;
  const size_t room = part_floats / (static_cast<size_t>(M) * 4);
  if (part == nullptr || room < 2) runs = 1;
  else if (static_cast<size_t>(runs) > room) runs = static_cast<int>(room);
  const int run = ((vocab + runs - 1) / runs + 3) / 4 * 4;
  runs = (vocab + run - 1) / run;
  HeadPart* hp = runs > 1 ? reinterpret_cast<HeadPart*>(part) : nullptr;
  const bool vec = vocab % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0;
  if (vec)
    hipLaunchKernelGGL(k_head_partial<true>, dim3(M, runs), dim3(kThreads), 0, st, logits, vocab, run, hp, rows,
                       n, L_p, sign, x0, conf);
  else
    hipLaunchKernelGGL(k_head_partial<false>, dim3(M, runs), dim3(kThreads), 0, st, logits, vocab, run, hp, rows,
                       n, L_p, sign, x0, conf);
  if (hp) launch_head_merge(hp, runs, M, rows, n, L_p, sign, x0, conf, st);
}

void launch_head_merge(const HeadPart* part, int n_part, int M, const int* rows, int n, int L_p, float sign,
                       int* x0, float* conf, hipStream_t st) {
  if (M <= 0) return;
  hipLaunchKernelGGL(k_head_merge, dim3(M), dim3(kThreads), 0, st, part, n_part, rows, n, L_p, sign, x0, conf);
}

void launch_apply_tokens(int* tokens, int B, int n, int L_p, const int* chosen, int chosen_stride,
                         int n_unmask, const int* x0, hipStream_t st) {
  const int total = B * n_unmask;
  if (total <= 0) return;
  hipLaunchKernelGGL(k_apply_tokens, dim3((total + kThreads - 1) / kThreads), dim3(kThreads), 0, st,
                     tokens, B, n, L_p, chosen, chosen_stride, n_unmask, x0);
}

}  // namespace dllmc
