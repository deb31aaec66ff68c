// Multi-head softmax attention over a packed qkv tensor [nb, S, 3D]
// (columns [Q|K|V], head h = columns h*dh..(h+1)*dh-1 of each third), no mask.
//
// Kernels on the fp32 matrix instructions for any element type, sequence length and head size (a multiple of 8,
// at most 128); bf16 with a head size of 64 has its own (attention_mfma.hip).  The backward pass recomputes the
// probabilities from the saved row log-sum-exp; no atomics, so results are reproducible.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace pt {

// ---------------------------------------------------------------------------
// Attention on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): fp32 mode, and bf16 with a head size other
// than 64 (widened to fp32 on the way in).  A wave owns 16 rows (queries, or keys of the dK / dV role), whose
// operands stay in registers; the other side streams through LDS in tiles of 64 rows, shared by four waves, the
// next tile's loads in flight while this one is multiplied.
//
// Scores are computed transposed where queries are owned, S^T = K Q^T, so that an accumulator holds the rows
// 4 g + v (g = lane / 16) of column lane % 16.  MFMA number v of the second product then takes register v as its
// operand as it stands, because the k index of a lane group is free as long as both operands agree: no probability
// goes through LDS, and the owned row of every accumulator is lane % 16, so that the softmax statistics are one
// value per lane and results leave in 16-byte pieces.
//
// What bounds it: the fp32 matrix rate.  The earlier kernels, plain FMA with every factor read from LDS, ran at 3
// TFLOP/s.  8 x 12 heads of 197 tokens, head size 64: forward 348 -> 24 us, backward 708 -> 64 us (one launch for
// both roles; the dK / dV workgroups take dO.O from the tiles they stage anyway).
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16* p) {
  union { uint2 u; bf16 h[4]; } t;
  t.u = *reinterpret_cast<const uint2*>(p);
  return f32x4{to_f32(t.h[0]), to_f32(t.h[1]), to_f32(t.h[2]), to_f32(t.h[3])};
}
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store4(bf16* p, f32x4 v) {
  union { uint2 u; bf16 h[4]; } t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t.h[i] = from_f32<bf16>(v[i]);
  *reinterpret_cast<uint2*>(p) = t.u;
}

constexpr int kAttnRows = 64;   // rows of a streamed tile, and rows owned by a workgroup of four waves

// DP: the head size rounded up to 16, 32, 64 or 128; columns from dh on are zeros
template <typename T, int DP>
struct AttnTile {
  static constexpr int LD = DP + 4;          // conflict-free for 16-byte reads of 16 rows and for single floats of 4 x 16
  static constexpr int FLOATS = kAttnRows * LD;
  static constexpr int N4 = DP / 16;         // pieces of four elements per thread
  static constexpr int NF = DP / 16;         // fragments of 16 columns
  static __device__ __forceinline__ void place(int tid, int i, int* row, int* d) {
    const int c = tid + 256 * i;
    *row = c / (DP / 4);
    *d = (c % (DP / 4)) * 4;
  }
  static __device__ __forceinline__ void load(const T* p, int64_t ld, int r0, int S, int dh, int tid, f32x4 (&reg)[N4]) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      int row, d;
      place(tid, i, &row, &d);
      reg[i] = r0 + row < S && d < dh ? load4(p + (int64_t)(r0 + row) * ld + d) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  static __device__ __forceinline__ void store(float* s, int tid, const f32x4 (&reg)[N4]) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      int row, d;
      place(tid, i, &row, &d);
      *reinterpret_cast<f32x4*>(s + row * LD + d) = reg[i];
    }
  }
  // an owned row's operand: lane group g holds columns 16 q + 4 g .. + 3 of row lane % 16
  static __device__ __forceinline__ void own(const T* p, int64_t ld, int row, int S, int dh, int g, float f, f32x4 (&reg)[NF]) {
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      const int d = 16 * q + 4 * g;
      reg[q] = row < S && d < dh ? load4(p + (int64_t)row * ld + d) * f : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // rows r0 + 0..15 of the tile times the owned rows, over the columns
  static __device__ __forceinline__ f32x4 dot(const float* s, int r0, int l, int g, const f32x4 (&own_)[NF]) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(s + (r0 + l) * LD + 16 * q + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], own_[q][e], acc, 0, 0, 0);
    }
    return acc;
  }
  // acc (columns 16 n + 4 g + v of the owned rows) += sum over rows r0 + 0..15 of tile row x weight
  static __device__ __forceinline__ void add(const float* s, int r0, int l, int g, f32x4 w, f32x4 (&acc)[NF]) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NF; ++n)
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(s[(r0 + 4 * g + v) * LD + 16 * n + l], w[v], acc[n], 0, 0, 0);
  }
  static __device__ __forceinline__ void put(T* p, int dh, int g, float f, const f32x4 (&acc)[NF]) {
#pragma unroll
    for (int n = 0; n < NF; ++n)
      if (16 * n + 4 * g < dh) store4(p + 16 * n + 4 * g, acc[n] * f);
  }
};

__device__ __forceinline__ float group_sum(float v) {   // over the four lane groups
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

template <typename T, int DP>
__global__ __launch_bounds__(256, DP > 64 ? 1 : 2) void attn_fwd_f32_kernel(const T* __restrict__ qkv, T* __restrict__ ctx,
                                                                             float* __restrict__ lse, int S, int H, int dh) {
  typedef AttnTile<T, DP> A;
  __shared__ __attribute__((aligned(16))) float xs[A::FLOATS], ys[A::FLOATS];
  const int D = H * dh, b = blockIdx.z, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int g = lane >> 4, l = lane & 15, row0 = blockIdx.x * kAttnRows + (tid >> 6) * 16, row = row0 + l;
  const T* base = qkv + (int64_t)b * S * 3 * D + h * dh;
  f32x4 q[A::NF], o[A::NF], rk[A::N4], rv[A::N4];
  A::own(base, 3 * D, row, S, dh, g, rsqrtf((float)dh), q);
#pragma unroll
  for (int n = 0; n < A::NF; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, sum = 0.f;   // sum: over this lane's own keys
  A::load(base + D, 3 * D, 0, S, dh, tid, rk);
  A::load(base + 2 * D, 3 * D, 0, S, dh, tid, rv);
  for (int k0 = 0; k0 < S; k0 += kAttnRows) {
    __syncthreads();
    A::store(xs, tid, rk);
    A::store(ys, tid, rv);
    __syncthreads();
    if (k0 + kAttnRows < S) {
      A::load(base + D, 3 * D, k0 + kAttnRows, S, dh, tid, rk);
      A::load(base + 2 * D, 3 * D, k0 + kAttnRows, S, dh, tid, rv);
    }
    if (row0 >= S) continue;   // a wave without rows only stages
    f32x4 s[4];
    float mx = m;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (k0 + 16 * u < S) {
        s[u] = A::dot(xs, 16 * u, l, g, q);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (k0 + 16 * u + 4 * g + v >= S) s[u][v] = -INFINITY;
          mx = fmaxf(mx, s[u][v]);
        }
      } else {
        s[u] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float ref = mx == -INFINITY ? 0.f : mx, alpha = __expf(m - ref);
    m = mx;
    sum *= alpha;
#pragma unroll
    for (int n = 0; n < A::NF; ++n) o[n] *= alpha;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (k0 + 16 * u >= S) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[u][v] = __expf(s[u][v] - ref);
        sum += s[u][v];
      }
      A::add(ys, 16 * u, l, g, s[u], o);
    }
  }
  if (row0 >= S) return;
  sum = group_sum(sum);
  if (row < S) {
    A::put(ctx + ((int64_t)b * S + row) * D + h * dh, dh, g, 1.0f / sum, o);
    if (lse && g == 0) lse[((int64_t)b * H + h) * S + row] = m + __logf(sum);
  }
}

// The probabilities are recomputed from the saved row log-sum-exp.  The first `tiles` workgroups of a head own 64
// queries each and stream K and V (dQ); the others own 64 keys and stream Q and dO (dK, dV): no atomics, every sum in
// a fixed order.
template <typename T, int DP>
__global__ __launch_bounds__(256, DP > 64 ? 1 : 2) void attn_bwd_f32_kernel(const T* __restrict__ qkv, const T* __restrict__ ctx,
                                                                             const T* __restrict__ dctx, const float* __restrict__ lse,
                                                                             T* __restrict__ dqkv, int S, int H, int dh, int tiles) {
  typedef AttnTile<T, DP> A;
  __shared__ __attribute__((aligned(16))) float xs[A::FLOATS], ys[A::FLOATS], ls[kAttnRows], dl[kAttnRows];
  const int D = H * dh, b = blockIdx.z, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const bool keys = (int)blockIdx.x >= tiles;
  const int g = lane >> 4, l = lane & 15;
  const int row0 = ((int)blockIdx.x - (keys ? tiles : 0)) * kAttnRows + (tid >> 6) * 16, row = row0 + l;
  const float scale = rsqrtf((float)dh);
  const T* base = qkv + (int64_t)b * S * 3 * D + h * dh;
  const T* obase = ctx + (int64_t)b * S * D + h * dh;
  const T* dobase = dctx + (int64_t)b * S * D + h * dh;
  const float* lrow = lse + ((int64_t)b * H + h) * S;
  T* out = dqkv + ((int64_t)b * S + row) * 3 * D + h * dh;
  f32x4 rx[A::N4], ry[A::N4], a0[A::NF], a1[A::NF], ax[A::NF];
#pragma unroll
  for (int n = 0; n < A::NF; ++n) ax[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (!keys) {
    A::own(base, 3 * D, row, S, dh, g, 1.f, a0);
    A::own(dobase, D, row, S, dh, g, 1.f, a1);
    float delta = 0.f;
    {
      f32x4 o[A::NF];
      A::own(obase, D, row, S, dh, g, 1.f, o);
#pragma unroll
      for (int n = 0; n < A::NF; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) delta = fmaf(a1[n][e], o[n][e], delta);
    }
    delta = group_sum(delta);
    const float lw = row < S ? lrow[row] : 0.f;
    A::load(base + D, 3 * D, 0, S, dh, tid, rx);
    A::load(base + 2 * D, 3 * D, 0, S, dh, tid, ry);
    for (int k0 = 0; k0 < S; k0 += kAttnRows) {
      __syncthreads();
      A::store(xs, tid, rx);
      A::store(ys, tid, ry);
      __syncthreads();
      if (k0 + kAttnRows < S) {
        A::load(base + D, 3 * D, k0 + kAttnRows, S, dh, tid, rx);
        A::load(base + 2 * D, 3 * D, k0 + kAttnRows, S, dh, tid, ry);
      }
      if (row0 >= S) continue;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + 16 * u >= S) continue;
        f32x4 s = A::dot(xs, 16 * u, l, g, a0);
        const f32x4 dp = A::dot(ys, 16 * u, l, g, a1);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          s[v] = k0 + 16 * u + 4 * g + v < S ? __expf(s[v] * scale - lw) * (dp[v] - delta) : 0.f;
        A::add(xs, 16 * u, l, g, s, ax);
      }
    }
    if (row < S) A::put(out, dh, g, scale, ax);
    return;
  }
  f32x4 ro[A::N4], ay[A::NF];
#pragma unroll
  for (int n = 0; n < A::NF; ++n) ay[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  A::own(base + D, 3 * D, row, S, dh, g, 1.f, a0);
  A::own(base + 2 * D, 3 * D, row, S, dh, g, 1.f, a1);
  A::load(base, 3 * D, 0, S, dh, tid, rx);
  A::load(dobase, D, 0, S, dh, tid, ry);
  A::load(obase, D, 0, S, dh, tid, ro);
  for (int q0 = 0; q0 < S; q0 += kAttnRows) {
    __syncthreads();
    A::store(xs, tid, rx);
    A::store(ys, tid, ry);
#pragma unroll
    for (int i = 0; i < A::N4; ++i) {   // DP / 4 neighbouring lanes hold a row
      int r, d;
      A::place(tid, i, &r, &d);
      float part = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) part = fmaf(ry[i][e], ro[i][e], part);
#pragma unroll
      for (int o = 1; o < DP / 4; o <<= 1) part += __shfl_xor(part, o, 64);
      if (d == 0) {
        dl[r] = part;
        ls[r] = q0 + r < S ? lrow[q0 + r] : INFINITY;   // rows past the end: probability exp(-inf) = 0
      }
    }
    __syncthreads();
    if (q0 + kAttnRows < S) {
      A::load(base, 3 * D, q0 + kAttnRows, S, dh, tid, rx);
      A::load(dobase, D, q0 + kAttnRows, S, dh, tid, ry);
      A::load(obase, D, q0 + kAttnRows, S, dh, tid, ro);
    }
    if (row0 >= S) continue;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (q0 + 16 * u >= S) continue;
      f32x4 p = A::dot(xs, 16 * u, l, g, a0);
      f32x4 ds = A::dot(ys, 16 * u, l, g, a1);
      const f32x4 lw = *reinterpret_cast<const f32x4*>(ls + 16 * u + 4 * g), dw = *reinterpret_cast<const f32x4*>(dl + 16 * u + 4 * g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = __expf(p[v] * scale - lw[v]);
        ds[v] = p[v] * (ds[v] - dw[v]);
      }
      A::add(ys, 16 * u, l, g, p, ay);
      A::add(xs, 16 * u, l, g, ds, ax);
    }
  }
  if (row < S) {
    A::put(out + D, dh, g, scale, ax);
    A::put(out + 2 * D, dh, g, 1.f, ay);
  }
}

template <typename T>
static void attention_fwd_t(const void* qkv, void* ctx, float* lse, int nb, int S, int H, int dh, hipStream_t st) {
  const dim3 grid(cdiv(S, kAttnRows), H, nb);
#define PT_F(DP_) hipLaunchKernelGGL((attn_fwd_f32_kernel<T, DP_>), grid, dim3(256), 0, st, (const T*)qkv, (T*)ctx, lse, S, H, dh)
  if (dh <= 16) PT_F(16);
  else if (dh <= 32) PT_F(32);
  else if (dh <= 64) PT_F(64);
  else PT_F(128);
#undef PT_F
}
template <typename T>
static void attention_bwd_t(const void* qkv, const void* ctx, const void* dctx, const float* lse, void* dqkv, int nb, int S,
                            int H, int dh, hipStream_t st) {
  const int tiles = cdiv(S, kAttnRows);
  const dim3 grid(2 * tiles, H, nb);
#define PT_B(DP_)                                                                                                          \
  hipLaunchKernelGGL((attn_bwd_f32_kernel<T, DP_>), grid, dim3(256), 0, st, (const T*)qkv, (const T*)ctx, (const T*)dctx, lse, \
                     (T*)dqkv, S, H, dh, tiles)
  if (dh <= 16) PT_B(16);
  else if (dh <= 32) PT_B(32);
  else if (dh <= 64) PT_B(64);
  else PT_B(128);
#undef PT_B
}

// 8 consecutive elements as floats / from floats (16-byte accesses for bf16)
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
  union { uint4 u; bf16 h[8]; } t;
  t.u = *reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = to_f32(t.h[i]);
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
  union { uint4 u; bf16 h[8]; } t;
#pragma unroll
  for (int i = 0; i < 8; ++i) t.h[i] = from_f32<bf16>(v[i]);
  *reinterpret_cast<uint4*>(p) = t.u;
}
// ---------------------------------------------------------------------------
// forward for each sample's first query only (the top block under a first-token head: no other row of its
// output is read).  One workgroup per (sample, head): s_t = scale q.k_t, p = softmax(s), o = sum_t p_t v_t.
// ctx_rows is dense: [nb, D]; the log-sum-exp goes to entry (b, h, 0) of the [nb, H, S] array the backward
// kernels read.  dh / 8 lanes share a key (whole rows are read); partial sums over keys are combined in
// a fixed order.
// ---------------------------------------------------------------------------
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void attn_fwd_first_query_kernel(const T* __restrict__ qkv, T* __restrict__ ctx_rows,
                                                                   float* __restrict__ lse, int S, int H, int dh) {
  extern __shared__ float sm[];
  float* qs = sm;            // [dh]
  float* sc = qs + dh;       // [S] scores, then unnormalised probabilities
  float* part = sc + S;      // [256 / (dh / 8)][dh] partial outputs of the key groups (VEC)
  __shared__ float red[4];
  const int D = H * dh;
  const int b = blockIdx.y, h = blockIdx.x, tid = threadIdx.x;
  const T* base = qkv + (int64_t)b * S * 3 * D + h * dh;
  const float scale = rsqrtf((float)dh);
  for (int d = tid; d < dh; d += 256) qs[d] = to_f32(base[d]);
  __syncthreads();
  const int lpr = VEC ? dh >> 3 : 1, j = tid % lpr, d0 = 8 * j, kpi = 256 / lpr;   // keys per iteration
  if (VEC) {
    for (int t0 = 0; t0 < S; t0 += kpi) {
      const int t = t0 + tid / lpr;
      const bool ok = t < S;
      float kv[8];
      load8(base + (int64_t)(ok ? t : 0) * 3 * D + D + d0, kv);
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) s = fmaf(qs[d0 + i], kv[i], s);
      for (int o = 1; o < lpr; o <<= 1) s += __shfl_xor(s, o, 64);
      if (ok && j == 0) sc[t] = s * scale;
    }
  } else {
    for (int t = tid; t < S; t += 256) {
      const T* kr = base + (int64_t)t * 3 * D + D;
      float s = 0.f;
      for (int d = 0; d < dh; ++d) s = fmaf(qs[d], to_f32(kr[d]), s);
      sc[t] = s * scale;
    }
  }
  __syncthreads();
  float lm = -INFINITY;
  for (int t = tid; t < S; t += 256) lm = fmaxf(lm, sc[t]);
  const float m = block_max<4>(lm, red);
  float ls = 0.f;
  for (int t = tid; t < S; t += 256) {
    const float p = __expf(sc[t] - m);
    sc[t] = p;
    ls += p;
  }
  const float l = block_sum<4>(ls, red);   // its barriers also publish sc
  const float inv = 1.0f / l;
  T* o = ctx_rows + (int64_t)b * D + h * dh;
  if (VEC) {
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    for (int t0 = 0; t0 < S; t0 += kpi) {
      const int t = t0 + tid / lpr;
      if (t < S) {
        float vv[8];
        load8(base + (int64_t)t * 3 * D + 2 * D + d0, vv);
        const float p = sc[t];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = fmaf(p, vv[i], acc[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) part[(tid / lpr) * dh + d0 + i] = acc[i];
    __syncthreads();
    for (int d = tid; d < dh; d += 256) {
      float a = 0.f;
      for (int g = 0; g < kpi; ++g) a += part[g * dh + d];
      o[d] = from_f32<T>(a * inv);
    }
  } else {
    for (int d = tid; d < dh; d += 256) {
      float a = 0.f;
      for (int t = 0; t < S; ++t) a = fmaf(sc[t], to_f32(base[(int64_t)t * 3 * D + 2 * D + d]), a);
      o[d] = from_f32<T>(a * inv);
    }
  }
  if (tid == 0 && lse) lse[((int64_t)b * H + h) * S] = m + __logf(l);
}
void attention_fwd_first_query(int dt, const void* qkv, void* ctx_rows, float* lse, int nb, int S, int H, int dh,
                               hipStream_t st) {
  if (nb <= 0) return;
  const bool vec = dh % 8 == 0 && 64 % (dh / 8) == 0 &&
                   (reinterpret_cast<uintptr_t>(qkv) | reinterpret_cast<uintptr_t>(ctx_rows)) % 16 == 0;
  const size_t shm = sizeof(float) * ((size_t)dh + S + (vec ? (size_t)(256 / (dh / 8)) * dh : 0));
#define PT_FQF(T, V)                                                                                                 \
  hipLaunchKernelGGL((attn_fwd_first_query_kernel<T, V>), dim3(H, nb), dim3(256), shm, st, (const T*)qkv, (T*)ctx_rows, \
                     lse, S, H, dh)
  if (dt == 0) { if (vec) PT_FQF(float, true); else PT_FQF(float, false); }
  else { if (vec) PT_FQF(bf16, true); else PT_FQF(bf16, false); }
#undef PT_FQF
}

// ---------------------------------------------------------------------------
// backward when only each sample's first query has a non-zero output gradient (the top block under a
// first-token head).  One workgroup per (sample, head): p_t = exp(q.k_t * scale - lse), dV_t = p_t dO,
// dS_t = p_t (dO.v_t - dO.o), dK_t = scale dS_t q, dQ_0 = scale sum_t dS_t k_t, dQ_t = 0 otherwise.
// ctx_rows and do_rows are dense: [nb, D], the first tokens' rows only.  One thread per key; the sum over
// keys for dQ_0 is taken by dh threads in key order (fixed, so reproducible).
// ---------------------------------------------------------------------------
// VEC: dh is a multiple of 8, so every head slice of a row starts on a 16-byte boundary and is moved in
// 8-element pieces
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void attn_bwd_first_query_kernel(const T* __restrict__ qkv, const T* __restrict__ ctx_rows,
                                                                   const T* __restrict__ do_rows,
                                                                   const float* __restrict__ lse, T* __restrict__ dqkv,
                                                                   int S, int H, int dh) {
  extern __shared__ float sm[];
  float* qs = sm;            // [dh]
  float* dos = qs + dh;      // [dh]
  float* dss = dos + dh;     // [S]
  __shared__ float delta_s;
  const int D = H * dh;
  const int b = blockIdx.y, h = blockIdx.x, tid = threadIdx.x;
  const T* base = qkv + (int64_t)b * S * 3 * D + h * dh;
  T* obase = dqkv + (int64_t)b * S * 3 * D + h * dh;
  const float scale = rsqrtf((float)dh);
  for (int d = tid; d < dh; d += 256) {
    qs[d] = to_f32(base[d]);
    dos[d] = to_f32(do_rows[(int64_t)b * D + h * dh + d]);
  }
  __syncthreads();
  if (tid == 0) {
    const T* o = ctx_rows + (int64_t)b * D + h * dh;
    float s = 0.f;
    for (int d = 0; d < dh; ++d) s = fmaf(dos[d], to_f32(o[d]), s);
    delta_s = s;
  }
  __syncthreads();
  const float l0 = lse[((int64_t)b * H + h) * S], dl = delta_s;
  float dqa_out[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    // dh / 8 lanes share a key: each moves one 16-byte piece of the key's rows, so a wave reads and writes
    // whole rows; the two dot products are finished with lane exchanges inside the group
    const int lpr = dh >> 3, j = tid % lpr, d0 = 8 * j, kpp = 256 / lpr;   // kpp keys per pass
    float dqa[8];   // this thread's share of dQ of the first token: sum over its keys of dS k
#pragma unroll
    for (int i = 0; i < 8; ++i) dqa[i] = 0.f;
    for (int t0 = 0; t0 < S; t0 += 4 * kpp) {   // four passes' rows in flight together
      float kv[4][8], vv[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + u * kpp + tid / lpr;
        const T* kr = base + (int64_t)(t < S ? t : 0) * 3 * D + D;
        load8(kr + d0, kv[u]);
        load8(kr + D + d0, vv[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + u * kpp + tid / lpr;
        float sc = 0.f, dp = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) { sc = fmaf(qs[d0 + i], kv[u][i], sc); dp = fmaf(dos[d0 + i], vv[u][i], dp); }
        for (int o = 1; o < lpr; o <<= 1) { sc += __shfl_xor(sc, o, 64); dp += __shfl_xor(dp, o, 64); }
        if (t < S) {
          const float pt = __expf(sc * scale - l0);
          const float ds = pt * (dp - dl);
          T* dq = obase + (int64_t)t * 3 * D;
          const float dsk = ds * scale;
          float z[8], a[8], c2[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            z[i] = 0.f; a[i] = dsk * qs[d0 + i]; c2[i] = pt * dos[d0 + i];
            dqa[i] = fmaf(ds, kv[u][i], dqa[i]);
          }
          if (t > 0) store8(dq + d0, z);
          store8(dq + D + d0, a);
          store8(dq + 2 * D + d0, c2);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) dqa_out[i] = dqa[i];
  } else {
    for (int t = tid; t < S; t += 256) {
      const T* kr = base + (int64_t)t * 3 * D + D;
      const T* vr = kr + D;
      float sc = 0.f, dp = 0.f;
      for (int d = 0; d < dh; ++d) { sc = fmaf(qs[d], to_f32(kr[d]), sc); dp = fmaf(dos[d], to_f32(vr[d]), dp); }
      const float pt = __expf(sc * scale - l0);
      const float ds = pt * (dp - dl);
      dss[t] = ds;
      T* dq = obase + (int64_t)t * 3 * D;
      T* dk = dq + D;
      T* dv = dk + D;
      const float dsk = ds * scale;
      for (int d = 0; d < dh; ++d) {
        if (t > 0) dq[d] = from_f32<T>(0.f);
        dk[d] = from_f32<T>(dsk * qs[d]);
        dv[d] = from_f32<T>(pt * dos[d]);
      }
    }
  }
  if (VEC) {
    // dQ of the first token: the threads' partial sums, combined in a fixed order (thread = pass slot * lpr + j)
    __shared__ float dqp[256 * 8];
    const int lpr = dh >> 3, kpp = 256 / lpr;
#pragma unroll
    for (int i = 0; i < 8; ++i) dqp[tid * 8 + i] = dqa_out[i];
    __syncthreads();
    for (int d = tid; d < dh; d += 256) {
      float acc = 0.f;
      for (int g = 0; g < kpp; ++g) acc += dqp[(g * lpr + (d >> 3)) * 8 + (d & 7)];
      obase[d] = from_f32<T>(acc * scale);
    }
    return;
  }
  __syncthreads();
  for (int d = tid; d < dh; d += 256) {
    float acc = 0.f;
    for (int t = 0; t < S; ++t) acc = fmaf(dss[t], to_f32(base[(int64_t)t * 3 * D + D + d]), acc);
    obase[d] = from_f32<T>(acc * scale);
  }
}
void attention_bwd_first_query(int dt, const void* qkv, const void* ctx_rows, const void* do_rows, const float* lse,
                               void* dqkv, int nb, int S, int H, int dh, hipStream_t st) {
  if (nb <= 0) return;
  const size_t shm = sizeof(float) * ((size_t)2 * dh + S);
  // the vector form needs 8 | dh, dh / 8 lanes per key dividing the wave, and 16-byte aligned tensors
  const bool vec = dh % 8 == 0 && 64 % (dh / 8) == 0 && (reinterpret_cast<uintptr_t>(qkv) | reinterpret_cast<uintptr_t>(dqkv)) % 16 == 0;
#define PT_FQ(T, V)                                                                                                   \
  hipLaunchKernelGGL((attn_bwd_first_query_kernel<T, V>), dim3(H, nb), dim3(256), shm, st, (const T*)qkv, (const T*)ctx_rows, \
                     (const T*)do_rows, lse, (T*)dqkv, S, H, dh)
  if (dt == 0) { if (vec) PT_FQ(float, true); else PT_FQ(float, false); }
  else { if (vec) PT_FQ(bf16, true); else PT_FQ(bf16, false); }
#undef PT_FQ
}

// matrix-core kernels for bf16, head size 64 (attention_mfma.hip)
void attention_fwd_mfma(const void* qkv, void* ctx, float* lse, int nb, int S, int H, hipStream_t st);
void attention_bwd_mfma(const void* qkv, const void* ctx, const void* dctx, const float* lse, void* dqkv, float* delta,
                        int nb, int S, int H, hipStream_t st);

// Longest sequence that a context with the fp32 kernels is accepted for.  The kernels stream any length; this is the
// supported range, the lengths whose scores for 32 queries and operand tiles fit 160 KB together.
int attention_f32_max_tokens(int dh) { return (1277 - 3 * dh) / 64 * 64; }
size_t attention_first_query_lds_bytes(int S, int dh) {
  const size_t fwd = sizeof(float) * ((size_t)dh + S + (dh % 8 == 0 ? (size_t)(256 / (dh / 8)) * dh : 0));
  const size_t bwd = sizeof(float) * ((size_t)2 * dh + S);
  return std::max(fwd, bwd);
}
bool attention_uses_mfma(int dt, int dh) { return dt == 1 && dh == 64; }

void attention_fwd(int dt, const void* qkv, void* ctx, float* lse, int nb, int S, int H, int dh, hipStream_t st) {
  if (nb <= 0) return;
  if (dt == 1 && dh == 64) { attention_fwd_mfma(qkv, ctx, lse, nb, S, H, st); return; }
  if (dt == 0) attention_fwd_t<float>(qkv, ctx, lse, nb, S, H, dh, st);
  else attention_fwd_t<bf16>(qkv, ctx, lse, nb, S, H, dh, st);
}

void attention_bwd(int dt, const void* qkv, const void* ctx, const void* dctx, const float* lse, void* dqkv,
                   float* delta_ws, int nb, int S, int H, int dh, hipStream_t st) {
  if (nb <= 0) return;
  if (dt == 1 && dh == 64) { attention_bwd_mfma(qkv, ctx, dctx, lse, dqkv, delta_ws, nb, S, H, st); return; }
  if (dt == 0) attention_bwd_t<float>(qkv, ctx, dctx, lse, dqkv, nb, S, H, dh, st);
  else attention_bwd_t<bf16>(qkv, ctx, dctx, lse, dqkv, nb, S, H, dh, st);
}

}  // namespace pt
