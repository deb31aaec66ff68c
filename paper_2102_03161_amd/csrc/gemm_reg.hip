// bf16 products with operands whose rows are even but no multiple of 8 elements long (MLP widths like 3076, patches of
// 14x14x3 = 588 values, class counts like 100), which the asynchronous global->LDS kernels cannot fetch in 16-byte
// pieces: forward products with such a width N, and weight gradients with such an M or N.
//
// Tiles go through registers: 16-byte loads along k of a k-major operand, pairs of rows of a strided one, transposed on
// their way to LDS, so that the operand reads of v_mfma_f32_32x32x16_bf16 are always 16 bytes.  What bounds it is the
// issue of those four-byte loads and the transposes.  Against 32x32 tiles of the fp32 instructions, unsplit:
// 12288 x 3076 x 768 with GELU 1452 -> 209 us, weight gradient 588 x 768 over 16384 tokens 772 -> 59 us.
#include <type_traits>
#include "common.h"
#include "kernels.h"
#include "gemm_epilogue.h"
#include "gemm_rules.h"

namespace pt {

namespace {

template <int BM_, int BN_, int BK_, int WGM_, int WGN_>
struct Cfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
  static constexpr int NT = 64 * WGM * WGN;          // threads
  static constexpr int WTM = BM / WGM, WTN = BN / WGN;  // per-wave tile
  static constexpr int TM = WTM / 32, TN = WTN / 32;    // 32x32 MFMA tiles per wave
  static constexpr int LDSK = BK + 8;  // padded rows: 16-byte operand reads of 8 consecutive rows hit distinct banks
  static constexpr int KC = BK / 8;    // 16-byte chunks per row
};

// Staging of one ROWS x BK operand tile in registers: NR dwords per thread.
// k-major operand (element (r,k) at p[r*ld + k]): 16-byte loads.
template <int ROWS, int BK, int NT>
struct KMajor {
  static constexpr int KC = BK / 8, CH = ROWS * KC / NT, NR = 4 * CH, LDSK = BK + 8;
  static_assert(ROWS * KC % NT == 0, "tile does not divide over the threads");
  static __device__ __forceinline__ void load(const bf16* p, int64_t ld, int R, int K, int r0, int k0, int tid,
                                              uint32_t (&reg)[NR]) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT;
      const int row = c / KC, kc = (c % KC) * 8;
      const int gr = r0 + row, gk = k0 + kc;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (gr < R && gk < K) v = *reinterpret_cast<const uint4*>(p + (int64_t)gr * ld + gk);
      reg[4 * i + 0] = v.x; reg[4 * i + 1] = v.y; reg[4 * i + 2] = v.z; reg[4 * i + 3] = v.w;
    }
  }
  static __device__ __forceinline__ void store(bf16* s, int tid, const uint32_t (&reg)[NR]) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT;
      const int row = c / KC, kc = (c % KC) * 8;
      *reinterpret_cast<uint4*>(s + row * LDSK + kc) = make_uint4(reg[4 * i], reg[4 * i + 1], reg[4 * i + 2], reg[4 * i + 3]);
    }
  }
};
// strided operand (element (r,k) at p[k*ld + r]): a task owns rows 2q,2q+1 and eight consecutive k;
// eight 4-byte loads (64 lanes cover 256 contiguous bytes), 2x2 16-bit transposes, two 16-byte LDS writes.
template <int ROWS, int BK, int NT>
struct Strided {
  static constexpr int QN = ROWS / 2, TASKS = QN * (BK / 8), TP = TASKS / NT, NR = 8 * TP, LDSK = BK + 8;
  static_assert(TASKS % NT == 0, "tile does not divide over the threads");
  static __device__ __forceinline__ void load(const bf16* p, int64_t ld, int R, int K, int r0, int k0, int tid,
                                              uint32_t (&reg)[NR]) {
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      const int t = tid + i * NT;
      const int q = t % QN, kg = t / QN;
      const int gr = r0 + 2 * q;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int gk = k0 + kg * 8 + j;
        reg[8 * i + j] = (gr < R && gk < K) ? *reinterpret_cast<const uint32_t*>(p + (int64_t)gk * ld + gr) : 0u;
      }
    }
  }
  static __device__ __forceinline__ void store(bf16* s, int tid, const uint32_t (&reg)[NR]) {
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      const int t = tid + i * NT;
      const int q = t % QN, kg = t / QN;
      const uint32_t* r = reg + 8 * i;
      uint4 even, odd;
      even.x = (r[0] & 0xffffu) | (r[1] << 16); odd.x = (r[0] >> 16) | (r[1] & 0xffff0000u);
      even.y = (r[2] & 0xffffu) | (r[3] << 16); odd.y = (r[2] >> 16) | (r[3] & 0xffff0000u);
      even.z = (r[4] & 0xffffu) | (r[5] << 16); odd.z = (r[4] >> 16) | (r[5] & 0xffff0000u);
      even.w = (r[6] & 0xffffu) | (r[7] << 16); odd.w = (r[6] >> 16) | (r[7] & 0xffff0000u);
      *reinterpret_cast<uint4*>(s + (2 * q) * LDSK + kg * 8) = even;
      *reinterpret_cast<uint4*>(s + (2 * q + 1) * LDSK + kg * 8) = odd;
    }
  }
  // column sums over k of the staged values: lo[i] += rows 2q, hi[i] += rows 2q+1
  static __device__ __forceinline__ void colsum(const uint32_t (&reg)[NR], float (&lo)[TP], float (&hi)[TP]) {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        lo[i] += __uint_as_float(reg[8 * i + j] << 16);
        hi[i] += __uint_as_float(reg[8 * i + j] & 0xffff0000u);
      }
  }
};

template <typename C, bool TA, int EPI, typename TC>
__global__ __launch_bounds__(C::NT, 4) void gemm_reg_kernel(GemmDev<bf16> g, SplitArgs sp, int tiles_n, int total_tiles,
                                                          int vec_ok) {
  typedef typename std::conditional<TA, Strided<C::BM, C::BK, C::NT>, KMajor<C::BM, C::BK, C::NT>>::type LA;
  typedef Strided<C::BN, C::BK, C::NT> LB;
  constexpr int LDSK = C::LDSK;
  constexpr int STAGE_LD = C::WTN + 4;
  constexpr int OPER_BYTES = 2 * (C::BM + C::BN) * LDSK * 2;
  constexpr int STAGE_BYTES = C::WGM * C::WGN * 32 * STAGE_LD * 4;
  constexpr int LDS_BYTES = OPER_BYTES > STAGE_BYTES ? OPER_BYTES : STAGE_BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];
  bf16* As = reinterpret_cast<bf16*>(lds);                       // [2][BM*LDSK]
  bf16* Bs = As + 2 * C::BM * LDSK;                              // [2][BN*LDSK]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / C::WGN, wn = wave % C::WGN;
  // Workgroups go round-robin to the 8 XCDs, each with its own L2: give every XCD a contiguous
  // run of tiles (n fastest) so that tiles sharing an A row panel meet in one L2.
  const int per = (total_tiles + 7) >> 3;
  const int lin = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (lin >= total_tiles) return;
  const int m0 = (lin / tiles_n) * C::BM, n0 = (lin % tiles_n) * C::BN;
  const int split = blockIdx.z;

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  uint32_t ra[LA::NR], rb[LB::NR];
  constexpr int CSN = LB::NR / 8;
  float cs_lo[CSN], cs_hi[CSN];
#pragma unroll
  for (int i = 0; i < CSN; ++i) { cs_lo[i] = 0.f; cs_hi[i] = 0.f; }
  const bool do_colsum = TA && sp.colsum != nullptr && m0 == 0;

  const int nk_all = (g.K + C::BK - 1) / C::BK;
  const int kt0 = split * sp.tiles_per_split;
  const int kt1 = (kt0 + sp.tiles_per_split < nk_all) ? kt0 + sp.tiles_per_split : nk_all;

  auto gload = [&](int kt) {
    LA::load(g.A, g.lda, g.M, g.K, m0, kt * C::BK, tid, ra);
    LB::load(g.B, g.ldb, g.N, g.K, n0, kt * C::BK, tid, rb);
    if (do_colsum) LB::colsum(rb, cs_lo, cs_hi);
  };
  auto sstore = [&](int buf) {
    LA::store(As + buf * C::BM * LDSK, tid, ra);
    LB::store(Bs + buf * C::BN * LDSK, tid, rb);
  };

  if (kt0 < kt1) {
    gload(kt0);
    sstore(0);
  }
  __syncthreads();
  int cur = 0;
  for (int kt = kt0; kt < kt1; ++kt) {
    if (kt + 1 < kt1) gload(kt + 1);
    const bf16* as = As + cur * C::BM * LDSK + (wm * C::WTM + (lane & 31)) * LDSK + (lane >> 5) * 8;
    const bf16* bs = Bs + cur * C::BN * LDSK + (wn * C::WTN + (lane & 31)) * LDSK + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < C::BK / 16; ++ks) {
      bf16x8 a[C::TM], b[C::TN];
#pragma unroll
      for (int i = 0; i < C::TM; ++i) a[i] = *reinterpret_cast<const bf16x8*>(as + i * 32 * LDSK + ks * 16);
#pragma unroll
      for (int j = 0; j < C::TN; ++j) b[j] = *reinterpret_cast<const bf16x8*>(bs + j * 32 * LDSK + ks * 16);
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < kt1) sstore(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }

  // ---- column sums of B (bias gradient riding on the weight-gradient product) ----
  if constexpr (TA) {
    if (do_colsum) {  // uniform over the workgroup; the main loop ended with a barrier
      float* red = reinterpret_cast<float*>(lds);  // [BK/8][BN]
#pragma unroll
      for (int i = 0; i < CSN; ++i) {
        const int t = tid + i * C::NT;
        const int q = t % (C::BN / 2), kg = t / (C::BN / 2);
        red[kg * C::BN + 2 * q] = cs_lo[i];
        red[kg * C::BN + 2 * q + 1] = cs_hi[i];
      }
      __syncthreads();
      for (int n = tid; n < C::BN; n += C::NT) {
        float s = 0.f;
#pragma unroll
        for (int kg = 0; kg < C::BK / 8; ++kg) s += red[kg * C::BN + n];
        if (n0 + n < g.N) sp.colsum[(int64_t)split * g.N + n0 + n] = s;
      }
      __syncthreads();
    }
  }

  void* Cbase = sizeof(TC) == 4 ? (void*)(reinterpret_cast<float*>(g.C) + split * sp.slab)
                                : (void*)(reinterpret_cast<bf16*>(g.C) + split * sp.slab);
  // one operand buffer: this kernel lives on having four small workgroups per CU
  staged_epilogue<C::TM, C::TN, C::WTM, C::WTN, EPI, TC, 1>(g, Cbase, acc, reinterpret_cast<float*>(lds) + wave * 32 * STAGE_LD,
                                                            m0 + wm * C::WTM, n0 + wn * C::WTN, lane, vec_ok);
}

template <typename C, bool TA, int EPI, typename TC>
void launch(const Gemm& a, int splits, float* cbase, int64_t slab, float* colsum_part, hipStream_t st) {
  GemmDev<bf16> g{(const bf16*)a.A, (const bf16*)a.B, cbase ? (void*)cbase : a.C, a.M, a.N, a.K, a.lda, a.ldb, a.ldc,
                  (const bf16*)a.bias, (const bf16*)a.aux, (bf16*)a.aux_out, a.ld_aux};
  const int tiles_m = cdiv(a.M, C::BM), tiles_n = cdiv(a.N, C::BN), total = tiles_m * tiles_n;
  const int nk = cdiv(a.K, C::BK);
  SplitArgs sp{splits, cdiv(nk, splits), slab, colsum_part};
  hipLaunchKernelGGL((gemm_reg_kernel<C, TA, EPI, TC>), dim3(8 * cdiv(total, 8), 1, splits), dim3(C::NT), 0, st, g, sp, tiles_n,
                     total, gemm_epilogue_vec_ok(a) ? 1 : 0);
}

template <typename C>
void dispatch(const Gemm& a, int splits, hipStream_t st) {
  if (!a.ta) {
    if (a.c_f32) launch<C, false, EPI_BIAS, float>(a, 1, nullptr, 0, nullptr, st);
    else launch<C, false, EPI_BIAS_GELU, bf16>(a, 1, nullptr, 0, nullptr, st);
    return;
  }
  // weight gradient: the bias gradient rides along as column sums of B
  const int64_t mn = (int64_t)a.M * a.N;
  float* cs_part = nullptr;
  if (a.colsum_out) cs_part = splits > 1 ? a.ws + splits * mn : a.colsum_out;
  launch<C, true, EPI_STORE, float>(a, splits, splits > 1 ? a.ws : nullptr, splits > 1 ? mn : 0, cs_part, st);
  if (splits > 1) gemm_splitk_reduce(a.ws, splits, mn, (float*)a.C, a.colsum_out ? cs_part : nullptr, a.N, a.colsum_out, st);
}

}  // namespace

void gemm_reg(const Gemm& a, hipStream_t st) {
  const GemmRegTiling t = gemm_reg_tiling(a);
  if (t.tile == 128) dispatch<Cfg<128, 128, 32, 2, 2>>(a, t.splits, st);
  else dispatch<Cfg<64, 64, 64, 2, 2>>(a, t.splits, st);
}

}  // namespace pt
