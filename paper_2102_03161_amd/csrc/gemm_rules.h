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

inline GemmPath gemm_path(int dt, const Gemm& a) {
  if (dt == 0 || !gemm_combo_used(a) || (a.ta && a.ldc != a.N)) return GEMM_F32;   // split-K slabs are dense
  if (gemm_dma_ok(a)) return GEMM_DMA;
  return gemm_reg_ok(a) ? GEMM_REG : GEMM_F32;
}

}  // namespace pt
