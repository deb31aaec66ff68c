// Products on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): every product of fp32 mode, and in bf16 mode
// those that neither bf16 kernel takes (k-major operands with a K that is no multiple of 8: the second MLP product and
// the first one's input gradient at such an MLP width, the patch embedding of 14x14x3 patches; odd or very small class
// counts); those operands are widened to fp32 on their way into LDS.
//
// What bounds it: the fp32 matrix rate (64 FLOP per clock and SIMD, 157 TFLOP/s on the chip) is a sixteenth of the
// bf16 one, so a 64x64 tile needs 38 GB/s of operands per CU where its load path carries 90 to 113; registers as
// staging and one k tile of lead are enough, and what counts is how evenly the 16x16 units of work fall on the
// 1024 SIMDs.  Four tile sizes serve that.  Operands lie in LDS as they lie in memory: an operand whose k runs
// contiguously as [row][BK + 4], read 16 bytes (four k) at a time, one whose rows run contiguously as
// [k][rows + 4], read one float at a time; both paddings are conflict-free for the sixteen-row fragments.
//
// MFMA number j of group q multiplies the k values 16 q + 4 g + j, g = 0..3: the same order for every layout and
// tile size, so that a row's result depends on neither.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "gemm_epilogue.h"
#include "gemm_rules.h"

namespace pt {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// four neighbouring elements, widened
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16* p) {
  union { uint2 u; bf16 h[4]; } t;
  t.u = *reinterpret_cast<const uint2*>(p);
  return f32x4{to_f32(t.h[0]), to_f32(t.h[1]), to_f32(t.h[2]), to_f32(t.h[3])};
}

constexpr int kMaxPlain = 4;
struct PlainProb {
  const void* A; const void* B; void* C;
  const void* bias; const void* aux; void* aux_out;
  float* colsum;              // column sums of B over k (strided B only), or null
  int64_t lda, ldb, ldc, ld_aux;
  int M, N, K, tile0, tiles_n;
};
struct PlainArgs {
  PlainProb p[kMaxPlain];
  int nprob, total, epi;
};

constexpr int kPlainBK = 32;

// one operand tile of ROWS rows and kPlainBK k values: N4 = ROWS / 32 pieces of four elements per thread
template <typename T, bool STRIDED, bool VEC, int ROWS>
struct PlainTile {
  static constexpr int N4 = ROWS / 32;
  static constexpr int LD = STRIDED ? ROWS + 4 : kPlainBK + 4;
  static constexpr int FLOATS = STRIDED ? kPlainBK * LD : ROWS * LD;
  static __device__ __forceinline__ void place(int tid, int i, int* row, int* k) {
    const int c = tid + 256 * i;
    if (STRIDED) { *k = c / (ROWS / 4); *row = (c % (ROWS / 4)) * 4; }
    else { *row = c / (kPlainBK / 4); *k = (c % (kPlainBK / 4)) * 4; }
  }
  static __device__ __forceinline__ void load(const T* p, int64_t ld, int R, int K, int r0, int k0, int tid, f32x4 (&reg)[N4]) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      int row, k;
      place(tid, i, &row, &k);
      row += r0; k += k0;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
        if (row < R && k < K) v = load4(p + (STRIDED ? (int64_t)k * ld + row : (int64_t)row * ld + k));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int re = STRIDED ? row + e : row, ke = STRIDED ? k : k + e;
          if (re < R && ke < K) v[e] = to_f32(p[STRIDED ? (int64_t)ke * ld + re : (int64_t)re * ld + ke]);
        }
      }
      reg[i] = v;
    }
  }
  static __device__ __forceinline__ void store(float* s, int tid, const f32x4 (&reg)[N4]) {
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      int row, k;
      place(tid, i, &row, &k);
      *reinterpret_cast<f32x4*>(s + (STRIDED ? k * LD + row : row * LD + k)) = reg[i];
    }
  }
  // the four k values 16 q + 4 g + j (j = 0..3) of row r
  static __device__ __forceinline__ f32x4 frag(const float* s, int r, int q, int g) {
    if (!STRIDED) return *reinterpret_cast<const f32x4*>(s + r * LD + 16 * q + 4 * g);
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = s[(16 * q + 4 * g + j) * LD + r];
    return v;
  }
};

// Column sums of B over k (the bias gradient of a weight-gradient product), from the fragments that the matrix
// instructions consume.  A column's k values go to four lanes, which add them in three levels: eight tiles (256 k), eight
// of those, the rest.  Relative error of that order on N(0, 1) columns: 9.9e-8 over 1576 tokens, 1.2e-7 over 12608
// (128 interleaved chains 1.3e-7 and 2.1e-7, one chain over all tokens 6.6e-7 and 2.0e-6).
template <int TN>
struct PlainColSum {
  float s0[TN], s1[TN], s2[TN];
  __device__ __forceinline__ PlainColSum() {
#pragma unroll
    for (int j = 0; j < TN; ++j) s0[j] = s1[j] = s2[j] = 0.f;
  }
  __device__ __forceinline__ void add(const f32x4 (&b)[TN]) {
#pragma unroll
    for (int j = 0; j < TN; ++j) s0[j] += (b[j][0] + b[j][1]) + (b[j][2] + b[j][3]);
  }
  // behind tile t
  __device__ __forceinline__ void fold(int t) {
    if ((t & 7) != 7) return;
#pragma unroll
    for (int j = 0; j < TN; ++j) { s1[j] += s0[j]; s0[j] = 0.f; }
    if ((t & 63) != 63) return;
#pragma unroll
    for (int j = 0; j < TN; ++j) { s2[j] += s1[j]; s1[j] = 0.f; }
  }
  // `out`: the sums of this wave's first column; n: columns that exist from there on
  __device__ __forceinline__ void store(float* out, int n, int lane) const {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float v = (s0[j] + s1[j]) + s2[j];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (lane < 16 && j * 16 + lane < n) out[j * 16 + lane] = v;
    }
  }
};

// Tiles of 32 TM x 32 TN, four waves in two rows of two, each TM x TN units of 16x16.  Up to four problems in one
// launch; workgroups go to the XCDs round-robin, and each XCD takes a contiguous run of tiles.
template <typename T, typename TC, bool TA, bool TB, bool VEC, int TM, int TN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(PlainArgs ga) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  typedef PlainTile<T, TA, VEC, BM> LA;
  typedef PlainTile<T, !TB, VEC, BN> LB;
  __shared__ __attribute__((aligned(16))) float lds[2 * (LA::FLOATS + LB::FLOATS)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int per = (ga.total + 7) >> 3;
  const int work = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (work >= ga.total) return;
  int pi = 0;
  while (pi + 1 < ga.nprob && work >= ga.p[pi + 1].tile0) ++pi;
  const PlainProb& p = ga.p[pi];
  const int local = work - p.tile0;
  const int m0 = (local / p.tiles_n) * BM, n0 = (local % p.tiles_n) * BN;
  const T* A = reinterpret_cast<const T*>(p.A);
  const T* B = reinterpret_cast<const T*>(p.B);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 ra[LA::N4], rb[LB::N4];
  const bool do_colsum = __builtin_amdgcn_readfirstlane(TA && p.colsum != nullptr && m0 == 0 && wm == 0 ? 1 : 0) != 0;
  PlainColSum<TN> cs;
  const int nk = (p.K + kPlainBK - 1) / kPlainBK;
  LA::load(A, p.lda, p.M, p.K, m0, 0, tid, ra);
  LB::load(B, p.ldb, p.N, p.K, n0, 0, tid, rb);
  for (int t = 0; t < nk; ++t) {
    float* as = lds + (t & 1) * (LA::FLOATS + LB::FLOATS);
    float* bs = as + LA::FLOATS;
    LA::store(as, tid, ra);
    LB::store(bs, tid, rb);
    __syncthreads();   // tile t is in LDS; the other buffer is free, its readers passed this barrier
    if (t + 1 < nk) {
      LA::load(A, p.lda, p.M, p.K, m0, (t + 1) * kPlainBK, tid, ra);
      LB::load(B, p.ldb, p.N, p.K, n0, (t + 1) * kPlainBK, tid, rb);
    }
    const int g = lane >> 4, l = lane & 15;
#pragma unroll
    for (int q = 0; q < kPlainBK / 16; ++q) {
      f32x4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = LA::frag(as, wm * 16 * TM + i * 16 + l, q, g);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = LB::frag(bs, wn * 16 * TN + j * 16 + l, q, g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
      if constexpr (TA) {
        if (do_colsum) cs.add(b);
      }
    }
    if constexpr (TA) {
      if (do_colsum) cs.fold(t);
    }
  }
  if constexpr (TA) {
    if (do_colsum) cs.store(p.colsum + n0 + wn * 16 * TN, p.N - n0 - wn * 16 * TN, lane);
  }
  // accumulator layout of the 16x16 MFMA: lane holds column lane % 16, rows 4 (lane / 16) + v
  const GemmDev<T> g{A, B, p.C, p.M, p.N, p.K, p.lda, p.ldb, p.ldc, reinterpret_cast<const T*>(p.bias),
                     reinterpret_cast<const T*>(p.aux), reinterpret_cast<T*>(p.aux_out), p.ld_aux};
  auto finish = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = m0 + (wm * TM + i) * 16 + 4 * (lane >> 4) + v, col = n0 + (wn * TN + j) * 16 + (lane & 15);
          if (row < p.M && col < p.N) epilogue_store<T, TC, EPI>(g, row, col, acc[i][j][v]);
        }
  };
  switch (ga.epi) {
    case EPI_STORE: finish(std::integral_constant<int, EPI_STORE>()); break;
    case EPI_BIAS: finish(std::integral_constant<int, EPI_BIAS>()); break;
    case EPI_BIAS_RES: finish(std::integral_constant<int, EPI_BIAS_RES>()); break;
    case EPI_BIAS_GELU: finish(std::integral_constant<int, EPI_BIAS_GELU>()); break;
    case EPI_MUL_DGELU: finish(std::integral_constant<int, EPI_MUL_DGELU>()); break;
    default: finish(std::integral_constant<int, EPI_RES>()); break;
  }
}

// pieces of four elements along the contiguous index
bool vec_ok(int dt, const Gemm& a) {
  const size_t bytes = dt == 0 ? 16 : 8;
  return aligned_to(a.A, bytes) && aligned_to(a.B, bytes) && a.lda % 4 == 0 && a.ldb % 4 == 0 && (a.ta ? a.M : a.K) % 4 == 0 &&
         (a.tb ? a.K : a.N) % 4 == 0;
}

template <typename T, typename TC, bool VEC, int TM, int TN>
void launch(const Gemm* a, int n, hipStream_t st) {
  PlainArgs ga{};
  int t0 = 0;
  for (int i = 0; i < n; ++i) {
    const Gemm& m = a[i];
    const int tiles_n = cdiv(m.N, 32 * TN);
    ga.p[i] = PlainProb{m.A, m.B, m.C, m.bias, m.aux, m.aux_out, m.colsum_out, m.lda, m.ldb, m.ldc, m.ld_aux,
                        m.M, m.N, m.K, t0, tiles_n};
    t0 += cdiv(m.M, 32 * TM) * tiles_n;
  }
  ga.nprob = n;
  ga.total = t0;
  ga.epi = a[0].epi;
  const dim3 grid(8 * cdiv(t0, 8));
  if (a[0].ta) hipLaunchKernelGGL((gemm_f32_kernel<T, TC, true, false, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
  else if (a[0].tb) hipLaunchKernelGGL((gemm_f32_kernel<T, TC, false, true, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
  else hipLaunchKernelGGL((gemm_f32_kernel<T, TC, false, false, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
}

template <bool VEC>
void choose_f32(const Gemm* a, int n, hipStream_t st) {
  const F32Tile t = gemm_f32_tile(a, n);
  if (t.tm == 4) launch<float, float, VEC, 4, 4>(a, n, st);
  else if (t.tm == 2) launch<float, float, VEC, 2, 2>(a, n, st);
  else if (t.tn == 2) launch<float, float, VEC, 1, 2>(a, n, st);
  else launch<float, float, VEC, 1, 1>(a, n, st);
}

// bf16 operands, widened: two tile sizes, the larger one from two workgroups per CU on (4096 x 768 x 3076 485 us on 32x32
// tiles with single-element loads, 257; 1024 rows 184 against 206), pieces of four where rows allow it (200 rows 139 -> 100 us)
template <typename TC>
void choose_bf16(const Gemm& a, hipStream_t st) {
  const bool vec = vec_ok(1, a), large = (int64_t)cdiv(a.M, 64) * cdiv(a.N, 64) >= 512;
  if (vec && large) launch<bf16, TC, true, 2, 2>(&a, 1, st);
  else if (vec) launch<bf16, TC, true, 1, 1>(&a, 1, st);
  else if (large) launch<bf16, TC, false, 2, 2>(&a, 1, st);
  else launch<bf16, TC, false, 1, 1>(&a, 1, st);
}

}  // namespace

void gemm_f32(int dt, const Gemm* a, int n, hipStream_t st) {
  if (dt != 0) {
    for (int i = 0; i < n; ++i) {
      if (a[i].c_f32) choose_bf16<float>(a[i], st);
      else choose_bf16<bf16>(a[i], st);
    }
    return;
  }
  for (int i = 0; i < n;) {
    int m = 1;   // products of one layout and epilogue over the same contraction share a launch
    while (m < kMaxPlain && i + m < n && a[i + m].ta == a[i].ta && a[i + m].tb == a[i].tb && a[i + m].epi == a[i].epi) ++m;
    bool vec = true;
    for (int j = 0; j < m; ++j) vec = vec && vec_ok(dt, a[i + j]);
    if (vec) choose_f32<true>(a + i, m, st);
    else choose_f32<false>(a + i, m, st);
    i += m;
  }
}

}  // namespace pt
