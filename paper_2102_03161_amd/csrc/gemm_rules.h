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
  if (a.lda >= (1 << 23) || a.ldb >= (1 << 23)) return false;   // 128 rows lie within 2^31 bytes: 32-bit offsets
  if (a.ta && (a.M % 8 || a.M < 8)) return false;      // strided operands: 16-byte pieces along the rows
  if (!a.tb && (a.N % 8 || a.N < 8)) return false;
  return (a.ta && !a.tb) || a.K % 8 == 0;              // a k-major operand: 16-byte pieces along k
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

// Variant of the asynchronous kernels, forward and input-gradient products: 1 = 128x128 tiles, 2 = 256x128, 3 = 64x64, 4 =
// 128x128 with eight waves, 5 / 6 = the two-group kernel with 256 / 192-row tiles, 7 = 128x64.  Every variant runs the same matrix
// instructions in the same k order, so a row's result does not depend on the choice (nor, through it, on the batch size).
inline int gemm_dma_variant(const Gemm& a) {
  auto cdiv = [](int64_t x, int64_t y) { return (x + y - 1) / y; };
  int pp = 0;   // the two-group kernel whose tiles fill the CUs well
  if (a.M >= 4096 && a.K % 64 == 0) {
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
    } else {
      const int v = cdiv(t192, 256) * 192 < cdiv(t256, 256) * 256 ? 6 : 5;
      // fewer tiles than 60 % of the CUs of their rounds (8192 tokens at N = 768: 129 tiles): smaller tiles fill the
      // chip better (6-13 % faster on those five products)
      const int64_t tiles = v == 6 ? t192 : t256;
      if (tiles * 10 >= cdiv(tiles, 256) * 256 * 6) pp = v;
    }
    if (pp && (a.M > 12288 || a.K < 256)) return pp;   // beyond what the cost lines below were fitted to
  }
  // Below that, 64x64, 128x64 or 128x128 tiles.  What bounds them is the way of the operands into LDS: the CU that gets the
  // most tiles brings in (rows + columns) * K of each, at 20 to 30 bytes per clock, and all CUs together share what the L2s
  // get from the memory side (loads alone take 20 of the 20.5 us of 1379 x 768 x 3072 on 64x64 tiles, and 14 when they
  // all hit the L2).
  const double k = 1e-3 * a.K;
  const int64_t t128 = cdiv(a.M, 128) * cdiv(a.N, 128), t64 = cdiv(a.M, 64) * cdiv(a.N, 64);
  // Forward products below 4096 rows keep to 64x64 and 128x128 tiles where 128x64 ones are fewer than 160 or do not all fit
  // (two to a CU): their weights come from beyond the L2s, which few workgroups fetch slowly.  In a step, 1379 x 768 x 768 and
  // 1379 x 768 x 3072 15.8 us on average on 64x64 tiles against 16.1 (alone 13.9 against 12.5), 2639 x 2304 x 768 17.2 on 128x128
  // ones against 17.8 (alone 17.4 against 16.4); input gradients 15.4 against 14.8.
  const int64_t t7 = cdiv(a.M, 128) * cdiv(a.N, 64);
  if (a.K % 64 || (!a.tb && a.M < 4096 && (t7 < 160 || t7 > 512))) {
    // Microseconds fitted to launches of 17 to 8192 rows with N and K of 768 to 3072, within 15 % (k = K / 1000): a 128x128
    // workgroup alone 5.7 + 8.9 k, w of them w (5.3 + 7.0 k); a 64x64 workgroup alone 3.5 + 4.7 k, w of them w (1.9 + 3.05 k).
    const double w128 = (double)((t128 + 255) / 256), w64 = (double)((t64 + 255) / 256);
    const double us128 = w128 > 1 ? w128 * (5.3 + 7.0 * k) : 5.7 + 8.9 * k;
    const double us64 = w64 > 1 ? w64 * (1.9 + 3.05 * k) : 3.5 + 4.7 * k;
    if (us64 <= us128) return 3;
    // K no multiple of 32: of the 128x128 tiles only eight waves on 64-wide k tiles take it (16384 x 1152 x 4304 228 us against 349 on 64x64
    // tiles and 235 on four waves with 32-wide ones; input gradients 254, 346, 273; 8192 x 3072 x 776 65, 98, 74)
    return a.K % 32 ? 4 : 1;
  }
  // Microseconds fitted to launches of 77 to 10400 rows with N and K of 256 to 4096, within 10 to 12 % (w: tiles on the
  // fullest CU).  1379 x 768 x 3072: 264 tiles of 64x64, 20.5 us, against 132 of 128x64, 18.0; 2639 x 768 x 3072 23.5 against
  // 19.5; 2639 x 3072 x 768 24.3 on 128x128 tiles against 25.6; 520 x 1024 x 4096 14.3 on 64x64 tiles against 20.9 on 128x64.
  // Over these launches the choice is 1.5 % off the fastest tile on average; with the two lines above alone it was 2.9 %.
  auto cost = [&](int bm, int bn, double one0, double one, double more0, double more, double load, double store) {
    const int64_t t = cdiv(a.M, bm) * cdiv(a.N, bn);
    return one0 + one * k + (double)(cdiv(t, 256) - 1) * (more0 + more * k) + load * 1e-8 * (double)t * (bm + bn) * a.K +
           store * 1e-6 * (double)a.M * a.N;
  };
  const double us64 = cost(64, 64, 3.07, 2.35, 0.1, 2.53, 2.69, 0.35), us128x64 = cost(128, 64, 3.33, 3.73, 0.7, 3.84, 3.64, 0.24);
  const double us128 = cost(128, 128, 4.24, 6.78, 2.09, 5.52, 7.24, 0.0);
  // eight waves and whole-line loads where both operands are k-major: 5-10 % faster where CUs hold two tiles
  const double us128x8 = a.tb ? cost(128, 128, 3.17, 8.44, 1.96, 4.15, 5.69, 0.22) : 1e30;
  struct Choice { int variant; double us; };
  const Choice small[4] = {{3, us64}, {7, us128x64}, {1, us128}, {4, us128x8}};
  Choice best = small[0];
  for (const Choice& c : small) if (c.us < best.us) best = c;
  if (a.M >= 4096) {
    // 5300 x 1536 x 384 21.7 us on 192x256 tiles, which fill 66 % of two rounds, against 17.1 on 128x128 ones; 5300 x 4096 x
    // 1024 (input gradient) 75.6 on 128x128 tiles against 63.9.  The lines are a few per cent off, so tiles that fill the CUs
    // well, and 128x128 ones (8192 x 768 x 3072 58.6 us, on 128x64 ones 61), have the benefit of the doubt.
    const double us256 = cost(256, 256, 5.74, 19.28, 12.33, 11.44, 3.69, 0.71), us192 = cost(192, 256, 5.98, 14.2, 19.37, 0.0, 7.65, 0.24);
    if (pp) return 0.93 * (pp == 5 ? us256 : us192) <= best.us ? pp : best.variant;
    if (us256 < best.us) best = Choice{5, us256};
    if (us192 < best.us) best = Choice{6, us192};
    const Choice square = us128x8 < us128 ? small[3] : small[2];
    if (0.85 * square.us <= best.us) best = square;
  }
  return best.variant;
}

// A block's weight gradients in one launch of the asynchronous kernels: square tiles (256: the two-group kernel, 64 and 128:
// the single-role pipeline) and the number of parts that the contraction is cut into, as far as the workspace of the
// first product has room for their slabs.
// Microseconds of a launch, fitted to launches over a block's four matrices of widths 256 and 768 with 231 to 12608
// tokens (within 15 %; k = tokens / 1000, s splits, w workgroups on the fullest CU):
//   64x64 tiles    the larger of 3.6 + 7.1 k / s (one workgroup's own chain) and w (1.2 + 3.75 k / s)
//   128x128 tiles  the larger of 4.7 + 12.5 k / s and w (4 + 9.8 k / s)
//   256x256 tiles  w (10 + 26 k / s)
// and for s > 1 the slabs' summation at 4 TB/s, also where it rides on another launch (WgradCarry).
// Width 768: 1379 tokens 34 us on 128x128 tiles against 43 on 64x64 ones, 2639 tokens 58 against 67 on 256x256 ones
// with two splits (a step of 2 x 2639 tokens, four blocks frozen, 5920 us against 6300), 8192 tokens 131 us on 256x256
// ones against 164 by the line above on 128x128; width 256: 231 tokens 5.2 us on 64x64 tiles, 2310 tokens 20 against
// 34 on 128x128 ones.
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
  for (int s = 1; s <= 4 && (s == 1 || a[0].K >= 512 * s); s *= 2) {
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
struct F32Tile { int tm, tn; };
inline F32Tile gemm_f32_tile(const Gemm* a, int n) {
  const double k = 1e-3 * a[0].K;
  struct Line { int tm, tn; double one0, one, more0, more, load, store; };
  static const Line lines[5] = {{1, 1, 2.85, 7.44, 0.11, 5.4, 0.0, 0.67}, {1, 2, 3.27, 11.37, 0.4, 9.87, 1.52, 0.43},
                                {2, 2, 3.72, 18.18, 0.18, 16.85, 5.75, 0.97}, {2, 3, 4.45, 26.08, 1.08, 24.85, 6.45, 0.79},
                                {4, 4, 6.49, 62.45, 0.0, 70.09, 7.21, 1.36}};
  F32Tile best{1, 1};
  double best_us = 1e300;
  for (const Line& l : lines) {
    int64_t t = 0;
    double out = 0.0;
    for (int i = 0; i < n; ++i) {
      t += (int64_t)((a[i].M + 32 * l.tm - 1) / (32 * l.tm)) * ((a[i].N + 32 * l.tn - 1) / (32 * l.tn));
      out += 1e-6 * (double)a[i].M * a[i].N;
    }
    const int64_t w = (t + 255) / 256;
    double us = l.one0 + l.one * k + (double)(w - 1) * (l.more0 + l.more * k) + l.load * 1e-8 * (double)t * 32 * (l.tm + l.tn) * a[0].K + l.store * out;
    if (l.tm == 4 && t * 10 >= w * 256 * 9) us *= 0.93;   // whole rounds of the largest tiles run a little ahead of the line
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
