// Products on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): every product of fp32 mode, and in bf16 mode
// those that neither bf16 kernel takes (k-major operands with a K that is no multiple of 8: the second MLP product and
// the first one's input gradient at such an MLP width, the patch embedding of 14x14x3 patches; odd or very small class
// counts); those operands are widened to fp32 on their way into LDS.
//
// What bounds it: the fp32 matrix rate (64 FLOP per clock and SIMD, 157 TFLOP/s on the chip) is a sixteenth of the
// bf16 one, so what counts is how evenly the 16x16 units of work fall on the 1024 SIMDs, and that a wave alone on its SIMD
// never waits between two halves of a k tile.  Five tile sizes serve the first (gemm_f32_tile).  gemm_f32_dma_kernel serves
// the second; it takes fp32 operands whose rows are 16-byte pieces.  The kernel that stages tiles through registers takes
// everything else: the operands lie in LDS as they lie in memory, an operand whose k runs contiguously as [row][BK + 4],
// read 16 bytes (four k) at a time, one whose rows run contiguously as [k][rows + 4], read one float at a time; both
// paddings are conflict-free for the sixteen-row fragments.
//
// MFMA number j of group q multiplies the k values 16 q + 4 g + j, g = 0..3: the same order for every kernel, layout and
// tile size, so that a row's result depends on none of them.
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
  int vec;                    // fp32 results and what the epilogue reads: 16-byte pieces
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
  // turns: column TN l + j is column l of unit j
  __device__ __forceinline__ void store(float* out, int n, int lane, bool turns = false) const {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float v = (s0[j] + s1[j]) + s2[j];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      const int col = turns ? TN * lane + j : j * 16 + lane;
      if (lane < 16 && col < n) out[col] = v;
    }
  }
};

// stores a wave's TM x TN units, whose first row and column are row0 and col0
template <typename T, typename TC, int TM, int TN>
__device__ __forceinline__ void f32_epilogue(const PlainProb& p, int epi_, int row0, int col0, int lane, const f32x4 (&acc)[TM][TN]) {
  // accumulator layout of the 16x16 MFMA: lane holds column lane % 16, rows 4 (lane / 16) + v
  const GemmDev<T> g{reinterpret_cast<const T*>(p.A), reinterpret_cast<const T*>(p.B), p.C, p.M, p.N, p.K, p.lda, p.ldb, p.ldc,
                     reinterpret_cast<const T*>(p.bias), reinterpret_cast<const T*>(p.aux), reinterpret_cast<T*>(p.aux_out), p.ld_aux};
  auto finish = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = row0 + i * 16 + 4 * (lane >> 4) + v, col = col0 + j * 16 + (lane & 15);
          if (row < p.M && col < p.N) epilogue_store<T, TC, EPI>(g, row, col, acc[i][j][v]);
        }
  };
  switch (epi_) {
    case EPI_STORE: finish(std::integral_constant<int, EPI_STORE>()); break;
    case EPI_BIAS: finish(std::integral_constant<int, EPI_BIAS>()); break;
    case EPI_BIAS_RES: finish(std::integral_constant<int, EPI_BIAS_RES>()); break;
    case EPI_BIAS_GELU: finish(std::integral_constant<int, EPI_BIAS_GELU>()); break;
    case EPI_MUL_DGELU: finish(std::integral_constant<int, EPI_MUL_DGELU>()); break;
    default: finish(std::integral_constant<int, EPI_RES>()); break;
  }
}

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
  f32_epilogue<T, TC, TM, TN>(p, ga.epi, m0 + wm * 16 * TM, n0 + wn * 16 * TN, lane, acc);
}

// ---- fp32 operands with 16-byte pieces: the same products through an asynchronous pipeline ----
// Operand tiles of 32 k values travel from global memory straight into LDS, three of them deep.  A k tile has two halves of
// 16 k; a half's MFMAs (512 clocks of a SIMD for 64x64 tiles) run while the next half's fragments are read into the other of
// two register sets, and the one barrier of a tile stands in front of its second half's MFMAs, where no wave has to wait for
// LDS.  Staged through registers, every tile had its LDS writes, barrier and fragment reads in a row in front of its MFMAs:
// 1576 x 768 x 3072 112 -> 87 us (86 TFLOP/s; 32x32 tiles), 231 x 768 x 3072 51 -> 27, 1576 x 2304 x 768 74 -> 64, 4081 x 1024 x
// 4096 354 -> 283 (121 TFLOP/s); a block's weight gradients at width 1024 over 1576 tokens 457 -> 362, at width 256 51 -> 34.
// With the reads in front of a half's MFMAs instead of between them the larger tiles are 5 to 7 % slower (4081 x 1024 x 4096
// 295); two or four tiles deep are the same within 3 %.
#define PT_LDS(p) ((__attribute__((address_space(3))) void*)(p))
#define PT_GLB(p) ((const __attribute__((address_space(1))) void*)(p))
// what lanes past the end of the contraction fetch
__device__ __attribute__((aligned(64))) const unsigned int f32_zeros[16] = {};

template <int N>
__device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }

// One operand tile.  k contiguous in memory: LDS image [ROWS][32], 128 bytes a row, 16-byte chunk c of row r in slot
// c ^ (r / 2 % 8); rows contiguous: image [32][ROWS], chunk c of row k in slot (c + 4 (k / 4 % 4)) mod (ROWS / 4), which
// keeps the four k groups of a fragment in different banks (two by two for 32 rows).
template <bool STRIDED, int ROWS>
struct DmaTile {
  static constexpr int LOADS = ROWS / 32, BYTES = ROWS * 128, UNITS = ROWS / 32;   // wave-wide loads per wave; 16-row units per wave
  static constexpr int CPR = STRIDED ? ROWS / 4 : 8;
  // A strided operand's two or four units take turns with the rows (row UNITS l + i is row l of unit i), so that one LDS read
  // brings all units' rows of one k: with a read per k and unit a block's weight gradients take 235 us instead of 224 (width 768,
  // 1576 tokens), 384 instead of 362 (width 1024).
  static constexpr bool TURNS = STRIDED && (UNITS == 2 || UNITS == 4);
  unsigned voff[LOADS];            // this lane's sources within a tile, bytes
  unsigned foff[TURNS ? 1 : STRIDED ? UNITS : 2];
  const char* src;                 // first byte of the tile that is loaded next
  int64_t step;
  static __device__ __forceinline__ int line(int wave, int i, int lane) { return (64 * (wave * LOADS + i) + lane) / CPR; }
  static __device__ __forceinline__ int chunk(int wave, int i, int lane) {
    const int slot = (64 * (wave * LOADS + i) + lane) % CPR, l = line(wave, i, lane);
    return STRIDED ? (slot + CPR - (4 * ((l >> 2) & 3)) % CPR) % CPR : slot ^ ((l >> 1) & 7);
  }
  static __device__ __forceinline__ int load_k(int wave, int i, int lane) {   // first k of the piece that this lane fetches
    return STRIDED ? line(wave, i, lane) : 4 * chunk(wave, i, lane);
  }
  // rows past the end are clamped to the last one (of a strided operand, to the last four): they feed outputs that are not stored
  __device__ __forceinline__ void setup(const float* p, int64_t ld, int R, int r0, unsigned lds0, int rbase, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      int r = STRIDED ? 4 * chunk(wave, i, lane) : line(wave, i, lane);
      const int k = load_k(wave, i, lane), last = R - (STRIDED ? 4 : 1) - r0;
      r = r < last ? r : last;
      voff[i] = 4u * (STRIDED ? (unsigned)k * (unsigned)ld + r : (unsigned)r * (unsigned)ld + k);
    }
    src = reinterpret_cast<const char*>(p + (STRIDED ? r0 : r0 * ld));
    step = STRIDED ? 128 * ld : 128;
    const int g = lane >> 4, l = lane & 15;
    if constexpr (STRIDED) {
#pragma unroll
      for (int i = 0; i < (TURNS ? 1 : UNITS); ++i) {
        const int r = TURNS ? rbase + UNITS * l : rbase + 16 * i + l;
        foff[i] = lds0 + 4 * g * ROWS * 4 + (((r >> 2) + 4 * g) % CPR) * 16 + (r & 3) * 4;
      }
    } else {
      const int r = rbase + l;
#pragma unroll
      for (int q = 0; q < 2; ++q) foff[q] = lds0 + r * 128 + (((4 * q + g) ^ ((r >> 1) & 7)) << 4);
    }
  }
  template <bool TAIL>
  __device__ __forceinline__ void issue(unsigned char* to, int wave, int klim) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const char* from = src + voff[i];
      if (TAIL && load_k(wave, i, threadIdx.x & 63) >= klim) from = reinterpret_cast<const char*>(f32_zeros);
      __builtin_amdgcn_global_load_lds(PT_GLB(from), PT_LDS(to + (wave * LOADS + i) * 1024), 16, 0, 0);
    }
    src += step;
  }
  // The k values 16 q + 4 g + j of every unit's rows, j = 0..3.  Inline assembly, because the compiler would wait for every
  // load into LDS in front of a read; the values are there behind arrived(), and nothing moves them before.
  struct Frag {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    // [k] with TURNS, else [unit][k] or a vector of four k per unit
    typename std::conditional<TURNS, typename std::conditional<UNITS == 2, f32x2, f32x4>::type[4],
                              typename std::conditional<STRIDED, float[UNITS][4], f32x4[UNITS]>::type>::type f;
    __device__ __forceinline__ float at(int i, int j) const {
      if constexpr (TURNS) return f[j][i];
      else return f[i][j];
    }
    __device__ __forceinline__ void arrived() {
      if constexpr (STRIDED && !TURNS) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(f[i][j]));
      } else {
#pragma unroll
        for (int i = 0; i < (TURNS ? 4 : UNITS); ++i) asm volatile("" : "+v"(f[i]));
      }
    }
  };
  static constexpr int READS = TURNS ? 4 : UNITS;   // parts that read() brings
  __device__ __forceinline__ void read(unsigned stage, int q, int i, Frag& to) const {
    if constexpr (TURNS) {
      const unsigned a = stage + foff[0];
      if constexpr (UNITS == 2) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(to.f[i]) : "v"(a), "n"((16 * q + i) * ROWS * 4));
      else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to.f[i]) : "v"(a), "n"((16 * q + i) * ROWS * 4));
    } else if constexpr (STRIDED) {
      const unsigned a = stage + foff[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(to.f[i][j]) : "v"(a), "n"((16 * q + j) * ROWS * 4));
    } else {
      const unsigned a = stage + foff[q];
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to.f[i]) : "v"(a), "n"(i * 16 * 128));
    }
  }
};

// Stores a wave's TM x TN units, whose first row and column are row0 and col0.  The matrix instructions got the operands the
// other way round, so a lane holds four neighbouring columns 4 (lane / 16) + v of row lane % 16 and moves 16 bytes at a
// time; one element at a time, 4081 x 3072 x 768 with GELU takes 231 us and 1576 x 3072 x 768 94.  vec: sizes and
// alignment allow it.
// TURNS_A, TURNS_B: whether the units take turns with the rows, the columns (DmaTile).
template <int TM, int TN, bool TURNS_A, bool TURNS_B>
__device__ __forceinline__ void f32_store(const PlainProb& p, int epi_, bool vec, int row0, int col0, int lane, const f32x4 (&acc)[TM][TN]) {
  const GemmDev<float> g{reinterpret_cast<const float*>(p.A), reinterpret_cast<const float*>(p.B), p.C, p.M, p.N, p.K, p.lda, p.ldb, p.ldc,
                         reinterpret_cast<const float*>(p.bias), reinterpret_cast<const float*>(p.aux), reinterpret_cast<float*>(p.aux_out), p.ld_aux};
  auto finish = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
    constexpr bool BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU;
    constexpr bool AUX = EPI == EPI_BIAS_RES || EPI == EPI_RES || EPI == EPI_MUL_DGELU;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = row0 + (TURNS_A ? TM * (lane & 15) + i : i * 16 + (lane & 15));
        const int col = col0 + (TURNS_B ? 4 * TN * (lane >> 4) + 4 * j : j * 16 + 4 * (lane >> 4));
        f32x4 v;   // four neighbouring columns: with turns, column TN u + j of the lane's 4 TN is element u of unit j
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = TURNS_B ? acc[i][(4 * j + e) % TN][(4 * j + e) / TN] : acc[i][j][e];
        if (row >= p.M || col >= p.N) continue;
        if (vec) {   // N is a multiple of four
          if (BIAS) {
            const f32x4 b = load4(g.bias + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += b[e];
          }
          if (AUX) {
            const f32x4 x = load4(g.aux + (int64_t)row * g.ld_aux + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = EPI == EPI_MUL_DGELU ? v[e] * x[e] : v[e] + x[e];
          }
          if (EPI == EPI_BIAS_GELU) {
            f32x4 dg;
#pragma unroll
            for (int e = 0; e < 4; ++e) { float d; v[e] = gelu_both(v[e], &d); dg[e] = d; }
            if (g.aux_out) *reinterpret_cast<f32x4*>(g.aux_out + (int64_t)row * g.ld_aux + col) = dg;
          }
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + (int64_t)row * g.ldc + col) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < p.N) epilogue_store<float, float, EPI>(g, row, col + e, v[e]);
        }
      }
  };
  switch (epi_) {
    case EPI_STORE: finish(std::integral_constant<int, EPI_STORE>()); break;
    case EPI_BIAS: finish(std::integral_constant<int, EPI_BIAS>()); break;
    case EPI_BIAS_RES: finish(std::integral_constant<int, EPI_BIAS_RES>()); break;
    case EPI_BIAS_GELU: finish(std::integral_constant<int, EPI_BIAS_GELU>()); break;
    case EPI_MUL_DGELU: finish(std::integral_constant<int, EPI_MUL_DGELU>()); break;
    default: finish(std::integral_constant<int, EPI_RES>()); break;
  }
}

// The same tiles, waves and order of k as gemm_f32_kernel.
template <bool TA, bool TB, int TM, int TN, int NS>
__global__ __launch_bounds__(256) void gemm_f32_dma_kernel(PlainArgs ga) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  typedef DmaTile<TA, BM> LA;
  typedef DmaTile<!TB, BN> LB;
  constexpr int STAGE = LA::BYTES + LB::BYTES, LPT = LA::LOADS + LB::LOADS;
  static_assert(NS >= 2 && NS <= 4 && NS * STAGE <= 160 * 1024 && LPT * (NS - 1) < 64, "LDS and vmcnt");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NS * STAGE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int per = (ga.total + 7) >> 3;
  const int work = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (work >= ga.total) return;
  int pi = 0;
  while (pi + 1 < ga.nprob && work >= ga.p[pi + 1].tile0) ++pi;
  const PlainProb& p = ga.p[pi];
  const int local = work - p.tile0;
  const int m0 = (local / p.tiles_n) * BM, n0 = (local % p.tiles_n) * BN;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool do_colsum = __builtin_amdgcn_readfirstlane(TA && p.colsum != nullptr && m0 == 0 && wm == 0 ? 1 : 0) != 0;
  PlainColSum<TN> cs;

  const int n = (p.K + kPlainBK - 1) / kPlainBK, klim = p.K - (n - 1) * kPlainBK;
  const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) const void*)lds);
  LA ta;
  LB tb;
  ta.setup(reinterpret_cast<const float*>(p.A), p.lda, p.M, m0, lds0, wm * 16 * TM, wave, lane);
  tb.setup(reinterpret_cast<const float*>(p.B), p.ldb, p.N, n0, lds0 + LA::BYTES, wn * 16 * TN, wave, lane);
  auto issue = [&](int t, int stage) {
    unsigned char* const to = lds + stage * STAGE;
    if (t == n - 1 && klim < kPlainBK) {
      ta.template issue<true>(to, wave, klim);
      tb.template issue<true>(to + LA::BYTES, wave, klim);
    } else {
      ta.template issue<false>(to, wave, kPlainBK);
      tb.template issue<false>(to + LA::BYTES, wave, kPlainBK);
    }
  };
  // at most the loads of the `later` youngest tiles are pending
  auto landed = [&](int later) {
    if (NS >= 4 && later >= 3) wait_vm<(NS >= 4 ? 3 : 0) * LPT>();
    else if (NS >= 3 && later >= 2) wait_vm<(NS >= 3 ? 2 : 0) * LPT>();
    else if (later >= 1) wait_vm<LPT>();
    else wait_vm<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  typename LA::Frag fa[2];
  typename LB::Frag fb[2];
  auto read = [&](int stage, int q, int u) {   // one part of the A fragments, then of the B fragments
    if (u < LA::READS) ta.read(stage * STAGE, q, u, fa[q]);
    else tb.read(stage * STAGE, q, u - LA::READS, fb[q]);
  };
  auto arrived = [&](int q) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fa[q].arrived();
    fb[q].arrived();
  };
  // The MFMAs of half q, and between the first of them the reads of the next half (of tile `stage`), so that the matrix cores
  // do not stand still while those are issued; `load` goes out behind the reads.
  auto half = [&](auto colsum, int q, int stage, auto load) {
    constexpr int COUNT = 4 * TM * TN, READS = LA::READS + LB::READS, EVERY = COUNT / 2 / READS < 1 ? 1 : COUNT / 2 / READS;   // within the first half of them
#pragma unroll
    for (int x = 0; x < COUNT; ++x) {
      const int e = x / (TM * TN), i = x / TN % TM, j = x % TN;
      if (x % EVERY == 0) {
        // the last MFMA takes what is left: small tiles have fewer MFMAs than reads
#pragma unroll
        for (int u = x / EVERY; u < READS && (u == x / EVERY || x + EVERY >= COUNT); ++u) read(stage, q ^ 1, u);
        __builtin_amdgcn_sched_barrier(0);
      }
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[q].at(j, e), fa[q].at(i, e), acc[i][j], 0, 0, 0);
      if (x == COUNT / 2) load();
    }
    if constexpr (decltype(colsum)::value) {
      f32x4 b[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = f32x4{fb[q].at(j, 0), fb[q].at(j, 1), fb[q].at(j, 2), fb[q].at(j, 3)};
      cs.add(b);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto run = [&](auto colsum) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s < n) issue(s, s);
    landed(n - 1 < NS - 1 ? n - 1 : NS - 1);
#pragma unroll
    for (int u = 0; u < LA::READS + LB::READS; ++u) read(0, 0, u);
    arrived(0);
    int cur = 0;
    for (int t = 0; t < n; ++t) {
      const int nxt = cur + 1 == NS ? 0 : cur + 1;
      half(colsum, 0, cur, []() {});
      arrived(1);
      // this wave is done with tile t's stage; behind the barrier everybody is, and tile t + 1 has landed
      const int later = n - 2 - t;
      landed(later < NS - 2 ? later : NS - 2);
      // behind the last tile the reads bring stale values that nothing multiplies
      half(colsum, 1, nxt, [&]() { if (t + NS < n) issue(t + NS, cur); });
      arrived(0);
      if constexpr (decltype(colsum)::value) cs.fold(t);
      cur = nxt;
    }
  };
  if (do_colsum) run(std::bool_constant<TA>());
  else run(std::false_type());
  if constexpr (TA) {
    if (do_colsum) cs.store(p.colsum + n0 + wn * 16 * TN, p.N - n0 - wn * 16 * TN, lane, LB::TURNS);
  }
  f32_store<TM, TN, LA::TURNS, LB::TURNS>(p, ga.epi, p.vec != 0, m0 + wm * 16 * TM, n0 + wn * 16 * TN, lane, acc);
}

// pieces of four elements along the contiguous index
bool vec_ok(int dt, const Gemm& a) {
  const size_t bytes = dt == 0 ? 16 : 8;
  return aligned_to(a.A, bytes) && aligned_to(a.B, bytes) && a.lda % 4 == 0 && a.ldb % 4 == 0 && (a.ta ? a.M : a.K) % 4 == 0 &&
         (a.tb ? a.K : a.N) % 4 == 0;
}

bool f32_out_vec_ok(const Gemm& m) {
  return m.N % 4 == 0 && m.ldc % 4 == 0 && aligned_to(m.C, 16) && (!m.bias || aligned_to(m.bias, 16)) &&
         ((!m.aux && !m.aux_out) || (m.ld_aux % 4 == 0 && aligned_to(m.aux, 16) && aligned_to(m.aux_out, 16)));
}

PlainArgs plain_args(const Gemm* a, int n, int bm, int bn) {
  PlainArgs ga{};
  int t0 = 0;
  for (int i = 0; i < n; ++i) {
    const Gemm& m = a[i];
    const int tiles_n = cdiv(m.N, bn);
    ga.p[i] = PlainProb{m.A, m.B, m.C, m.bias, m.aux, m.aux_out, m.colsum_out, m.lda, m.ldb, m.ldc, m.ld_aux,
                        m.M, m.N, m.K, t0, tiles_n, f32_out_vec_ok(m) ? 1 : 0};
    t0 += cdiv(m.M, bm) * tiles_n;
  }
  ga.nprob = n;
  ga.total = t0;
  ga.epi = a[0].epi;
  return ga;
}

template <typename T, typename TC, bool VEC, int TM, int TN>
void launch(const Gemm* a, int n, hipStream_t st) {
  const PlainArgs ga = plain_args(a, n, 32 * TM, 32 * TN);
  const dim3 grid(8 * cdiv(ga.total, 8));
  if (a[0].ta) hipLaunchKernelGGL((gemm_f32_kernel<T, TC, true, false, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
  else if (a[0].tb) hipLaunchKernelGGL((gemm_f32_kernel<T, TC, false, true, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
  else hipLaunchKernelGGL((gemm_f32_kernel<T, TC, false, false, VEC, TM, TN>), grid, dim3(256), 0, st, ga);
}

template <int TM, int TN, int NS>
void launch_dma(const Gemm* a, int n, hipStream_t st) {
  const PlainArgs ga = plain_args(a, n, 32 * TM, 32 * TN);
  const dim3 grid(8 * cdiv(ga.total, 8));
  if (a[0].ta) hipLaunchKernelGGL((gemm_f32_dma_kernel<true, false, TM, TN, NS>), grid, dim3(256), 0, st, ga);
  else if (a[0].tb) hipLaunchKernelGGL((gemm_f32_dma_kernel<false, true, TM, TN, NS>), grid, dim3(256), 0, st, ga);
  else hipLaunchKernelGGL((gemm_f32_dma_kernel<false, false, TM, TN, NS>), grid, dim3(256), 0, st, ga);
}

void choose_f32(const Gemm* a, int n, bool vec, hipStream_t st) {
  const F32Tile t = gemm_f32_tile(a, n, vec);
  if (vec) {
    if (t.tm == 4) launch_dma<4, 4, 3>(a, n, st);
    else if (t.tn == 3) launch_dma<2, 3, 3>(a, n, st);
    else if (t.tm == 2) launch_dma<2, 2, 3>(a, n, st);
    else if (t.tn == 2) launch_dma<1, 2, 3>(a, n, st);
    else launch_dma<1, 1, 3>(a, n, st);
    return;
  }
  if (t.tm == 4) launch<float, float, false, 4, 4>(a, n, st);
  else if (t.tm == 2) launch<float, float, false, 2, 2>(a, n, st);
  else if (t.tn == 2) launch<float, float, false, 1, 2>(a, n, st);
  else launch<float, float, false, 1, 1>(a, n, st);
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
    for (int j = 0; j < m; ++j) vec = vec && vec_ok(dt, a[i + j]) && a[i + j].K >= 1 && a[i + j].lda < (1 << 22) && a[i + j].ldb < (1 << 22);   // 128 rows within 2^31 bytes
    choose_f32(a + i, m, vec, st);
    i += m;
  }
}

}  // namespace pt
