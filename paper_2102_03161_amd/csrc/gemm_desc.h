// A dense product C = epilogue(A x B) as its callers describe it.  Plain C++: the choice of a kernel (gemm_rules.h) is
// tested without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace pt {

enum Epi {
  EPI_STORE = 0,      // C = acc
  EPI_BIAS = 1,       // C = acc + bias[n]
  EPI_BIAS_RES = 2,   // C = acc + bias[n] + aux[m,n]
  EPI_BIAS_GELU = 3,  // h = acc + bias[n]; aux_out[m,n] = GELU'(h) (if non-null); C = GELU(h)
  EPI_MUL_DGELU = 4,  // C = acc * aux[m,n], aux = the GELU'(h) that EPI_BIAS_GELU saved
  EPI_RES = 5         // C = acc + aux[m,n]
};

struct Gemm {
  const void* A = nullptr;  // ta ? [K,M] : [M,K], leading dimension lda
  const void* B = nullptr;  // tb ? [N,K] : [K,N], leading dimension ldb
  void* C = nullptr;        // [M,N], leading dimension ldc; T, or float when c_f32
  int M = 0, N = 0, K = 0;
  int64_t lda = 0, ldb = 0, ldc = 0;
  bool ta = false, tb = false;
  Epi epi = EPI_STORE;
  const void* bias = nullptr;  // T [N]
  const void* aux = nullptr;   // T [M,N] ld_aux (fp32 when c_f32: the gradient stream)
  void* aux_out = nullptr;     // T [M,N] ld_aux
  int64_t ld_aux = 0;
  bool c_f32 = false;
  // weight-gradient products (ta && !tb, fp32 C with ldc == N) may split K over several workgroups
  // through `ws` (ws_floats fp32 of scratch) and can also return the column sums of B over K
  // (the bias gradient) in colsum_out[N]
  float* ws = nullptr;
  size_t ws_floats = 0;
  float* colsum_out = nullptr;
};

}  // namespace pt
