// Dense contractions of the encoder block, C = epilogue(A x B): which kernel a product goes to, and the summation of
// split-K slabs.
//
//  * gemm_dma.hip: bf16 operands on the bf16 matrix cores, global->LDS pipelines.
//  * gemm_reg.hip: bf16 operands on the bf16 matrix cores, rows that are even but no multiple of 8 elements long.
//  * gemm_f32.hip: fp32 mode, and what is left of bf16 operands, on the fp32 matrix cores.
//
// Forward and input-gradient products run their K loop in a fixed order without split-K (but for the few-row
// products of an active top block), so every output element is a deterministic function of its own row and column.
#include <algorithm>
#include "common.h"
#include "kernels.h"
#include "gemm_epilogue.h"
#include "gemm_rules.h"

namespace pt {

// A second, short vector (the column-sum partials of the same product) may ride along in the last workgroups.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int splits, int64_t n,
                                                            float* __restrict__ out, int vec, int blocks_main,
                                                            const float* __restrict__ part2, int64_t n2,
                                                            float* __restrict__ out2, int vec2) {
  if ((int)blockIdx.x < blocks_main) {
    splitk_sum4(part, splits, n, out, vec, ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4);
  } else {
    const int64_t i = ((int64_t)(blockIdx.x - blocks_main) * 256 + threadIdx.x) * 4;
    if (i < n2) splitk_sum4(part2, splits, n2, out2, vec2, i);
  }
}

int splitk_vec_ok4(const float* part, int64_t n, const float* out) {
  return (n % 4 == 0 && (reinterpret_cast<uintptr_t>(part) % 16) == 0 && (reinterpret_cast<uintptr_t>(out) % 16) == 0) ? 1 : 0;
}
static int vec_ok4(const float* part, int64_t n, const float* out) { return splitk_vec_ok4(part, n, out); }
void gemm_splitk_reduce(const float* part, int splits, int64_t n, float* out, const float* part2, int64_t n2, float* out2,
                        hipStream_t st) {
  const int blocks_main = (int)cdiv64(n, 1024);
  const int blocks2 = part2 ? (int)cdiv64(n2, 1024) : 0;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(blocks_main + blocks2)), dim3(256), 0, st, part, splits, n, out,
                     vec_ok4(part, n, out), blocks_main, part2, part2 ? n2 : 0, out2, part2 ? vec_ok4(part2, n2, out2) : 0);
}

// the reductions of up to four products in one launch (same split count)
struct ReduceGroup {
  const float* part[4]; float* out[4]; int64_t n[4]; int vec[4];
  const float* part2[4]; float* out2[4]; int64_t n2[4]; int vec2[4];
  int block0[5];      // first workgroup of each product
  int blocks_main[4];
  int nprob, splits;
};
__global__ __launch_bounds__(256) void splitk_reduce_group_kernel(ReduceGroup rg) {
  int p = 0;
  while (p + 1 < rg.nprob && (int)blockIdx.x >= rg.block0[p + 1]) ++p;
  const int b = (int)blockIdx.x - rg.block0[p];
  if (b < rg.blocks_main[p]) {
    splitk_sum4(rg.part[p], rg.splits, rg.n[p], rg.out[p], rg.vec[p], ((int64_t)b * 256 + threadIdx.x) * 4);
  } else {
    const int64_t i = ((int64_t)(b - rg.blocks_main[p]) * 256 + threadIdx.x) * 4;
    if (i < rg.n2[p]) splitk_sum4(rg.part2[p], rg.splits, rg.n2[p], rg.out2[p], rg.vec2[p], i);
  }
}
void gemm_splitk_reduce_group(int nprob, int splits, const float* const* part, const int64_t* n, float* const* out,
                              const float* const* part2, const int64_t* n2, float* const* out2, hipStream_t st) {
  ReduceGroup rg{};
  rg.nprob = nprob;
  rg.splits = splits;
  int b0 = 0;
  for (int i = 0; i < nprob; ++i) {
    rg.part[i] = part[i]; rg.out[i] = out[i]; rg.n[i] = n[i]; rg.vec[i] = vec_ok4(part[i], n[i], out[i]);
    rg.part2[i] = part2[i]; rg.out2[i] = out2[i]; rg.n2[i] = part2[i] ? n2[i] : 0;
    rg.vec2[i] = part2[i] ? vec_ok4(part2[i], n2[i], out2[i]) : 0;
    rg.block0[i] = b0;
    rg.blocks_main[i] = (int)cdiv64(n[i], 1024);
    b0 += rg.blocks_main[i] + (part2[i] ? (int)cdiv64(n2[i], 1024) : 0);
  }
  rg.block0[nprob] = b0;
  hipLaunchKernelGGL(splitk_reduce_group_kernel, dim3((unsigned)b0), dim3(256), 0, st, rg);
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
// 16-byte epilogue accesses need 8-element alignment of everything the epilogue touches
bool gemm_epilogue_vec_ok(const Gemm& a) {
  bool ok = a.N % 8 == 0 && a.ldc % 8 == 0 && aligned_to(a.C, 16);
  if (a.bias) ok = ok && aligned_to(a.bias, 16);
  if (a.aux) ok = ok && a.ld_aux % 8 == 0 && aligned_to(a.aux, 16);
  if (a.aux_out) ok = ok && a.ld_aux % 8 == 0 && aligned_to(a.aux_out, 16);
  return ok;
}

bool gemm_uses_mfma(int dt, const Gemm& a) { return gemm_path(dt, a) != GEMM_F32; }

void gemm(int dt, const Gemm& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return;
  if (a.c_f32 && (a.epi == EPI_BIAS_GELU || a.epi == EPI_MUL_DGELU)) return;  // not used by the step
  const GemmPath path = gemm_path(dt, a);
  if (path == GEMM_REG) { gemm_reg(a, st); return; }
  if (path == GEMM_DMA) {
    if (!a.ta) {
      if (!gemm_dma_skinny(a, st)) gemm_dma(a, gemm_dma_variant(a), st);
      return;
    }
    // a weight gradient alone: 256x128 tiles (128x128 for small outputs) split over a long K, otherwise one
    // group of its own
    if (a.K % 32 == 0 && a.K >= 2048) { gemm_dma(a, (int64_t)a.M * a.N <= 1024 * 1024 ? 1 : 2, st); return; }
    if (gemm_wgrad_group(&a, 1, st, nullptr, nullptr, nullptr)) return;
  }
  gemm_f32(dt, &a, 1, st);
}

void gemm_wgrad_flush(WgradCarry* carry, hipStream_t st) {
  if (!carry || carry->nprob <= 0) return;
  gemm_splitk_reduce_group(carry->nprob, carry->splits, carry->part, carry->n, carry->out, carry->part2, carry->n2,
                           carry->out2, st);
  carry->nprob = 0;
}

void gemm_wgrad_batch(int dt, const Gemm* g, int n, hipStream_t st, hipEvent_t mid, WgradCarry* carry, LnBwdRide* ln) {
  if (ln) ln->taken_np = 0;
  if (n <= 0) return;
  if (dt == 0) { gemm_f32(dt, g, n, st); if (mid) (void)hipEventRecord(mid, st); return; }
  bool mfma = true;
  for (int i = 0; i < n && mfma; ++i) mfma = gemm_uses_mfma(dt, g[i]);
  // one product alone goes to the grouped kernel too when its contraction is long (the tokens of a batch)
  if (mfma && (n > 1 || g[0].K >= 2048) && gemm_wgrad_group(g, n, st, mid, carry, ln)) return;
  gemm_wgrad_flush(carry, st);
  for (int i = 0; i < n; ++i) gemm(dt, g[i], st);
  if (mid) (void)hipEventRecord(mid, st);
}

}  // namespace pt
