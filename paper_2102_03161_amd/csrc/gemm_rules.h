// Which kernel a product goes to: functions of its sizes, strides and alignment alone.  Plain C++, so that a test
// can ask for the choice without a GPU.
#pragma once
#include <algorithm>
#include "gemm_desc.h"

namespace pt {

enum GemmPath {
  GEMM_F32 = 0,   // gemm_f32.hip: the fp32 matrix instructions, any sizes and strides
  GEMM_REG = 1,   // gemm_reg.hip: bf16 matrix instructions, tiles staged through registers
  GEMM_DMA = 2    // gemm_dma.hip: bf16 matrix instructions, global->LDS pipelines
};

inline bool aligned_to(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// whether (layout, epilogue, output type) is one of the combinations the training step uses
inline bool gemm_combo_used(const Gemm& a) {
  if (a.ta && a.tb) return false;
  if (a.ta) return a.c_f32 && a.epi == EPI_STORE;                                             // weight gradient
  if (a.tb) return a.c_f32 ? (a.epi == EPI_RES || a.epi == EPI_STORE) : (a.epi == EPI_STORE || a.epi == EPI_MUL_DGELU);  // input gradient
  return a.c_f32 ? (a.epi == EPI_BIAS || a.epi == EPI_BIAS_RES)                                 // forward
                 : (a.epi == EPI_BIAS || a.epi == EPI_BIAS_RES || a.epi == EPI_BIAS_GELU);
}

// what the asynchronous kernels need: 16-byte pieces of every operand
inline bool gemm_dma_ok(const Gemm& a) {
  if (!aligned_to(a.A, 16) || !aligned_to(a.B, 16) || a.lda % 8 || a.ldb % 8 || a.K < 1) return false;
  if (a.ta && (a.M % 8 || a.M < 8)) return false;      // strided operands: 16-byte pieces along the rows
  if (!a.tb && (a.N % 8 || a.N < 8)) return false;
  return (a.ta && !a.tb) || a.K % 8 == 0;              // a k-major operand: 16-byte pieces along k
}

// What the lean k loop needs besides (64-column tiles, small weight gradients): a tile's rows, at most 128 of a k-major operand
// and 64 of a strided one, within the 2^32 bytes that a lane's unsigned offset spans.  Only the head's products over the first
// tokens of long sequences have rows far enough apart.
inline bool gemm_lean_ok(const Gemm& a) {
  auto within = [](bool k_major, int64_t rows, int64_t ld) { return ((k_major ? std::min<int64_t>(rows, 128) : 64) - 1) * ld * 2 + 256 < ((int64_t)1 << 32); };
  return within(!a.ta, a.M, a.lda) && within(a.tb, a.N, a.ldb);
}

// What the register-staged kernel needs: 16-byte pieces along k of a k-major operand, pairs along the rows of a
// strided one.  The row count of a forward or input-gradient product is not asked, so that a row's result does not
// depend on the batch it comes in.
inline bool gemm_reg_ok(const Gemm& a) {
  const bool a_ok = a.ta ? (a.M >= 32 && a.M % 2 == 0 && a.lda % 2 == 0 && aligned_to(a.A, 4))
                         : (a.K % 8 == 0 && a.lda % 8 == 0 && aligned_to(a.A, 16));
  const bool b_ok = a.tb ? (a.K % 8 == 0 && a.ldb % 8 == 0 && aligned_to(a.B, 16))
                         : (a.N % 2 == 0 && a.ldb % 2 == 0 && aligned_to(a.B, 4));
  // what the step has of such rows; weight gradients over a handful of tokens only write (768 x 3076 over 24 tokens: 9
  // us on the fp32 instructions' smaller tiles, 12 here; over 200 tokens 35 against 16)
  const bool used = a.ta ? a.K > 32 : (a.c_f32 ? a.epi == EPI_BIAS : a.epi == EPI_BIAS_GELU);
  return used && !a.tb && a_ok && b_ok && a.N >= 32;
}

// Its tiles (128 or 64 square) and, for weight gradients, the number of parts of K: few output tiles and a long
// contraction are split into fp32 slabs of the workspace, which are then added in a fixed order.  Four small workgroups
// fit a CU either way, so 128 wins once the launch is several times that: 768 x 3076 with 1024 rows 32 us on 64x64
// tiles against 44, with 2048 rows 54 against 50; weight gradient 3076 x 768 over 1024 tokens 25 against 31, over 4096
// 99 against 86; 588 x 768 over 4096 tokens 25 against 29, over 16384 69 against 60.
struct GemmRegTiling { int tile, splits; };
inline GemmRegTiling gemm_reg_tiling(const Gemm& a) {
  const int64_t t128 = (int64_t)((a.M + 127) / 128) * ((a.N + 127) / 128), t64 = (int64_t)((a.M + 63) / 64) * ((a.N + 63) / 64);
  if (!a.ta) return GemmRegTiling{t128 >= 384 ? 128 : 64, 1};
  const int tile = t128 * a.K >= 400000 ? 128 : 64;
  int64_t splits = 1;
  if (a.ws) {   // at least eight (four) k tiles of 32 (64) in a part
    splits = std::min<int64_t>(tile == 128 ? 768 / t128 : 1024 / t64, (a.K + 31) / 32 / 8);
    splits = std::max<int64_t>(std::min<int64_t>(splits, 16), 1);
    while (splits > 1 && (size_t)(splits * ((int64_t)a.M * a.N + a.N)) > a.ws_floats) --splits;
  }
  return GemmRegTiling{tile, (int)splits};
}

// 64x64 tiles: the kernel with four stages.  One workgroup on a CU has three tiles in flight instead of two: 1344 x 768 x 3072
// 15.4 -> 13.1 us, 231 x 768 x 3072 13.4 -> 11.1, 900 x 1024 x 1024 6.6 -> 6.0 (launches in a loop, weights in the L2s); with more
// than one the third workgroup that fits beside 48 KB counts for more (1379 x 3072 x 768 17.7 -> 19.6), and a short K has nothing
// to hide (231 x 256 x 256 3.7 -> 3.9).
inline bool gemm_64_four_stages(const Gemm& a) {
  return (int64_t)((a.M + 63) / 64) * ((a.N + 63) / 64) <= 256 && a.K >= 512;
}

// Variant of the asynchronous kernels, forward and input-gradient products: 1 = 128x128 tiles, 2 = 256x128, 3 = 64x64, 4 =
// 128x128 with eight waves, 5 / 6 = the two-group kernel with 256 / 192-row tiles, 7 = 128x64.  Every variant runs the same matrix
// instructions in the same k order, so a row's result does not depend on the choice (nor, through it, on the batch size).
inline int gemm_dma_variant(const Gemm& a) {
  auto cdiv = [](int64_t x, int64_t y) { return (x + y - 1) / y; };
  const double k = 1e-3 * a.K;
  const bool lean = gemm_lean_ok(a);
  if (a.K % 64) {
    // 64x64 or 128x128 tiles.  Microseconds fitted to launches of 17 to 8192 rows with N and K of 768 to 3072 (k = K / 1000): a
    // 128x128 workgroup alone 5.7 + 8.9 k, w of them w (5.3 + 7.0 k); a 64x64 workgroup alone 3.5 + 4.7 k, w of them
    // w (1.9 + 3.05 k).  The 64x64 lines are those of an older k loop, up to a third above the present one; over 722 products of
    // widths 200 to 1152 and 17 to 16384 rows the choice is 1.7 % off the fastest tile on average (10 to 28 % for 62 of them,
    // 10000 x 600 x 2400 the worst).
    const int64_t t128 = cdiv(a.M, 128) * cdiv(a.N, 128), t64 = cdiv(a.M, 64) * cdiv(a.N, 64);
    const double w128 = (double)((t128 + 255) / 256), w64 = (double)((t64 + 255) / 256);
    const double us128 = w128 > 1 ? w128 * (5.3 + 7.0 * k) : 5.7 + 8.9 * k;
    const double us64 = w64 > 1 ? w64 * (1.9 + 3.05 * k) : 3.5 + 4.7 * k;
    if (lean && us64 <= us128) return 3;
    // K no multiple of 32: of the 128x128 tiles only eight waves on 64-wide k tiles take it (16384 x 1152 x 4304 228 us against 349 on 64x64
    // tiles and 235 on four waves with 32-wide ones; input gradients 254, 346, 273; 8192 x 3072 x 776 65, 98, 74)
    return a.K % 32 ? 4 : 1;
  }
  int pp = 0;   // the two-group kernel whose tiles fill the CUs well
  if (a.M >= 4096) {
    // At least 4096 rows: the two-group kernel with 256x256 or 192x256 tiles, one workgroup per CU, whichever
    // fills whole rounds of 256 CUs better (M = 12608, N = 768: 198 tiles of 192x256 against 150 of 256x256).
    const int64_t tn = cdiv(a.N, 256);
    const int64_t t192 = cdiv(a.M, 192) * tn, t256 = cdiv(a.M, 256) * tn;
    if (a.N >= 3072 && (a.K < 1024 || a.tb)) {
      // Wide and short: 192- or 256-row tiles only when their last round is (nearly) full, as for 12288 tokens
      // (768 tiles of 192 rows at N = 3072; 9-10 % faster than 256x128 there) or 25216 (1188 tiles of 256 rows, 93 %
      // of five rounds: 169 us against 183 with GELU, 149 against 164 with the saved GELU'); otherwise from 9000
      // rows on 256x128 tiles, two workgroups per CU, whose prologues and epilogues overlap.
      const int64_t last = t192 % 256;
      if (last == 0 || last >= 224) pp = 6;
      else if (t256 * 10 >= cdiv(t256, 256) * 256 * 9) pp = 5;
      else if (a.M >= 9000) return 2;
      else if (t256 * 10 >= cdiv(t256, 256) * 256 * 8) pp = 5;   // 4400 x 3072 x 768 36.7 us, 44.3 on 128x128 tiles
    } else {
      const int v = cdiv(t192, 256) * 192 < cdiv(t256, 256) * 256 ? 6 : 5;
      // fewer tiles than 60 % of the CUs of their rounds (8192 tokens at N = 768: 129 tiles): smaller tiles fill the
      // chip better (6-13 % faster on those five products)
      const int64_t tiles = v == 6 ? t192 : t256;
      if (tiles * 10 >= cdiv(tiles, 256) * 256 * 6) pp = v;
    }
    if (pp && (a.M > 16384 || a.K < 256)) return pp;   // beyond what their lines below were fitted to
  }
  // What bounds the smaller tiles is the way of the operands into LDS: the CU that gets the most tiles brings in (rows +
  // columns) * K of each, at 20 to 30 bytes per clock, and all CUs together share what comes from beyond the L2s.  A line per
  // tile: a workgroup alone, each further one on the fullest of 256 CUs, all loads, the stores, and each further round of as
  // many as a CU holds at a time.  The constants were fitted to the choice between the lines, and only roughly to
  // microseconds, over 1645 products of 17 to 28000 rows, widths of 256 to 1280 and MLPs four times as wide, timed the way a
  // step runs them: the weights come from HBM (600 MB of them in turn), the other operand is recent.  There the choice is 0.3 %
  // off the fastest of its tiles on average below 4096 rows and 0.6 % up to 16384 (lines fitted to launches with their weights
  // in the L2s: 1.4 and 4.2 %); more than 5 % off are 37 of 1642 products, more than 10 % only 4400 to 5300 x 1024 x 4096 (84
  // on 128x128 tiles, 66 to 70 on 128x64) and 11500 x 1024 x 256.  Forward, us: 4000 x 768 x 3072 36.5 on 64x64 tiles, 31.9 on
  // 128x64, 40.7 on 128x128; 1379 x 3072 x 768 18.5, 19.8, 20.6; 4600 x 512 x 2048 23.6, 21.8, 29.2; 6500 x 768 x 3072 58.2, 54.2,
  // 50.5; input gradient 8192 x 3072 x 768 74.8, 65.6, 62.8, with eight waves 53.9.
  auto cost = [&](int bm, int bn, int held, double one0, double one, double more0, double more, double load, double store, double round) {
    const int64_t t = cdiv(a.M, bm) * cdiv(a.N, bn), w = cdiv(t, 256);
    return one0 + one * k + (double)(w - 1) * (more0 + more * k) + load * 1e-8 * (double)t * (bm + bn) * a.K + store * 1e-6 * (double)a.M * a.N +
           (double)(cdiv(w, held) - 1) * round * k;
  };
  struct Choice { int variant; double us; };
  Choice best{1, cost(128, 128, 3, 4.48, 9.69, 3.25, 2.11, 5.50, 0.03, 3.94)};
  auto consider = [&](int variant, double us) { if (us < best.us) best = Choice{variant, us}; };
  if (lean) {
    consider(3, gemm_64_four_stages(a) ? cost(64, 64, 2, 2.97, 3.76, 0.0, 0.0, 1.26, 0.38, 0.0)
                                       : cost(64, 64, 3, 2.57, 2.52, 0.64, 1.15, 7.16, 0.0, 1.16));
    consider(7, cost(128, 64, 2, 3.21, 5.73, 0.95, 2.08, 1.56, 0.28, 5.38));
  }
  // Eight waves with whole-line loads where both operands are k-major.  A step with forward products on them (8192 x 3072 x 768
  // and 8192 x 768 x 3072, alone within 1 % of four waves) was 0.5 % slower.
  if (a.tb) consider(4, cost(128, 128, 2, 2.41, 13.19, 0.99, 0.02, 3.06, 0.45, 6.08));
  if (pp == 5) consider(5, cost(256, 256, 1, 17.80, 10.06, 13.11, 11.52, 2.98, 0.05, 0.37));
  if (pp == 6) consider(6, cost(192, 256, 1, 10.83, 16.12, 20.17, 0.0, 0.01, 0.01, 0.03));
  return best.variant;
}

// A block's weight gradients in one launch of the asynchronous kernels: square tiles (256: the two-group kernel, 64 and 128:
// the single-role pipeline) and the number of parts that the contraction is cut into, as far as the workspace of the
// first product has room for their slabs.
// Microseconds of a launch (k = tokens / 1000, s splits, w workgroups on the fullest CU):
//   64x64 tiles    the larger of 3.6 + 7.1 k / s (one workgroup's own chain) and w (1.2 + 3.75 k / s)
//   128x128 tiles  the larger of 4.7 + 12.5 k / s and w (4 + 9.8 k / s)
//   256x256 tiles  w (10 + 26 k / s)
// and for s > 1 the slabs' summation at 4 TB/s, also where it rides on another launch (WgradCarry).
// The lines were fitted at widths 256 and 768 (231 to 12608 tokens, within 15 %) to an older k loop of the two smaller tiles.
// Of the present kernels, at widths 128 to 1280 and 17 to 16384 tokens, with the first operand from HBM, they are off by 12 %
// on average for 128 and 256, 21 % for 64x64 tiles (up to 63 %), and say too much by 7 to 18 % for split launches.  The
// choice suffers less: 1.5 % off the fastest on average over 262 such launches, more than 5 % for 29 of them.  The worst are
// width 384 from 4096 tokens on (6500 tokens 57 us on 64x64 tiles, 44 on 128x128 ones with four splits), width 512 from 4096 to
// 4400 (61, on 256x256 tiles 51) and width 768 from 4400 to 5500 (98 to 85 on 256x256 tiles, which also carry the passes that ride
// there, 93 to 77 on 128x128 ones).
// Width 768, alone: 1379 tokens 31 us on 128x128 tiles, 47 on 64x64 ones; 2639 tokens 50, on 256x256 ones with two splits 61;
// 8192 tokens 126 on 256x256 ones, 134 on 128x128.  Width 256: 231 tokens 5.4 us on 64x64 tiles, 7.3 on 128x128; 2310 tokens
// 16 to 17, on 128x128 18 to 27.
struct WgradTiling { int tile, splits; };
inline WgradTiling wgrad_tiling(const Gemm* a, int n) {
  const double k = 1e-3 * a[0].K;
  int64_t floats = 0, per_split = 0;
  for (int i = 0; i < n; ++i) {
    floats += (int64_t)a[i].M * a[i].N;
    per_split += (int64_t)a[i].M * a[i].N + a[i].N;
  }
  auto tiles = [&](int b) {
    int64_t t = 0;
    for (int i = 0; i < n; ++i) t += (int64_t)((a[i].M + b - 1) / b) * ((a[i].N + b - 1) / b);
    return t;
  };
  WgradTiling best{64, 1};
  double best_us = 1e30;
  auto consider = [&](int b, int s, double chain0, double chain, double each0, double each) {
    const double w = (double)((tiles(b) * s + 255) / 256);
    double us = std::max(chain0 + chain * k / s, w * (each0 + each * k / s));
    if (s > 1) us += 4.0 + (s + 1) * floats * 1e-6;
    if (us < best_us) { best_us = us; best = WgradTiling{b, s}; }
  };
  bool lean = true;
  for (int i = 0; i < n; ++i) lean = lean && gemm_lean_ok(a[i]);
  for (int s = 1; lean && s <= 4 && (s == 1 || a[0].K >= 512 * s); s *= 2) {
    consider(64, s, 3.6, 7.1, 1.2, 3.75);
    consider(128, s, 4.7, 12.5, 4.0, 9.8);
  }
  const int s = (int)std::min<int64_t>(std::min<int64_t>(256 / tiles(256), a[0].K / 256), 16);
  consider(256, s < 1 ? 1 : s, 10.0, 26.0, 10.0, 26.0);
  while (best.splits > 1 && (size_t)(best.splits * per_split) > a[0].ws_floats) --best.splits;
  return best;
}
// workspace floats that a block's four weight gradients (D x 3D, D x D, D x F, F x D) may use
inline size_t gemm_wgrad_batch_ws_floats(int D, int F) {
  const int64_t shapes[4][2] = {{D, 3 * D}, {D, D}, {D, F}, {F, D}};
  int64_t tiles = 0, per_split = 0;
  for (auto& sh : shapes) {
    tiles += ((sh[0] + 255) / 256) * ((sh[1] + 255) / 256);
    per_split += sh[0] * sh[1] + sh[1];
  }
  const int64_t splits = std::min<int64_t>(16, std::max<int64_t>(1, 256 / std::max<int64_t>(tiles, 1)));
  return (size_t)(splits * per_split);
}

// Tiles of a launch of up to four products on the fp32 matrix instructions, in units of 32 rows and columns.  Microseconds
// fitted to launches of 17 to 8000 rows (weight gradients: tokens) with widths of 64 to 4096 in all three layouts, within 5 to
// 8 % (k = K / 1000, w: tiles on the fullest CU): a k tile's MFMAs, once for each tile that shares the SIMDs, the loads of
// all tiles, the stores.  The choice is 0.7 % off the fastest tile on average.  1576 x 768 x 768: 1200 tiles of 32x32 25 us,
// 300 of 64x64 33; 4081 x 768 x 3072: 512 of 64x96 176 us, 768 of 64x64 181, 3072 of 32x32 224; 4081 x 1024 x 4096: 256 of
// 128x128 279 us, 1024 of 64x64 324.
// pipeline false: the kernel that stages its tiles through registers, element by element (rows that are no 16-byte pieces: odd
// patches and class counts), with lines of its own, fitted to 492 forward products, input and weight gradients of such sizes;
// the choice is 0.3 % off the fastest tile on average, by the pipeline's lines 1.6 % (6400 x 256 x 363 37 us on 32x32 tiles, 29 on
// 64x64).
struct F32Tile { int tm, tn; };
inline F32Tile gemm_f32_tile(const Gemm* a, int n, bool pipeline = true) {
  const double k = 1e-3 * a[0].K;
  struct Line { int tm, tn; double one0, one, more0, more, load, store; };
  static const Line piped[5] = {{1, 1, 2.85, 7.44, 0.11, 5.4, 0.0, 0.67}, {1, 2, 3.27, 11.37, 0.4, 9.87, 1.52, 0.43},
                                {2, 2, 3.72, 18.18, 0.18, 16.85, 5.75, 0.97}, {2, 3, 4.45, 26.08, 1.08, 24.85, 6.45, 0.79},
                                {4, 4, 6.49, 62.45, 0.0, 70.09, 7.21, 1.36}};
  static const Line staged[4] = {{1, 1, 2.73, 16.07, 0.07, 9.0, 6.59, 1.29}, {1, 2, 3.51, 24.75, 0.67, 10.98, 16.55, 0.13},
                                 {2, 2, 4.21, 39.4, 0.75, 20.55, 11.82, 0.59}, {4, 4, 6.82, 98.64, 0.04, 79.47, 1.35, 1.39}};
  F32Tile best{1, 1};
  double best_us = 1e300;
  for (int j = 0; j < (pipeline ? 5 : 4); ++j) {
    const Line& l = pipeline ? piped[j] : staged[j];
    int64_t t = 0;
    double out = 0.0;
    for (int i = 0; i < n; ++i) {
      t += (int64_t)((a[i].M + 32 * l.tm - 1) / (32 * l.tm)) * ((a[i].N + 32 * l.tn - 1) / (32 * l.tn));
      out += 1e-6 * (double)a[i].M * a[i].N;
    }
    const int64_t w = (t + 255) / 256;
    double us = l.one0 + l.one * k + (double)(w - 1) * (l.more0 + l.more * k) + l.load * 1e-8 * (double)t * 32 * (l.tm + l.tn) * a[0].K + l.store * out;
    if (pipeline && l.tm == 4 && t * 10 >= w * 256 * 9) us *= 0.93;   // whole rounds of the largest tiles run a little ahead of the line
    if (us < best_us) { best_us = us; best = F32Tile{l.tm, l.tn}; }
  }
  return best;
}

inline GemmPath gemm_path(int dt, const Gemm& a) {
  if (dt == 0 || !gemm_combo_used(a) || (a.ta && a.ldc != a.N)) return GEMM_F32;   // split-K slabs are dense
  if (gemm_dma_ok(a)) return GEMM_DMA;
  return gemm_reg_ok(a) ? GEMM_REG : GEMM_F32;
}

}  // namespace pt
