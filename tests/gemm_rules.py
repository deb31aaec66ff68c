"""The library's choice of a kernel for a product (csrc/gemm_rules.h), compiled for the host and asked through ctypes."""
import ctypes
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_03161_amd", "csrc")

F32, REG, DMA = 0, 1, 2                                     # GemmPath
STORE, BIAS, BIAS_RES, BIAS_GELU, MUL_DGELU, RES = range(6)  # Epi

SOURCE = r"""
#include "gemm_rules.h"
using namespace pt;
static Gemm make(int M, int N, int K, int ta, int tb, int epi, int c_f32, long long ws_floats) {
  Gemm g;
  g.A = g.B = g.C = reinterpret_cast<void*>(uintptr_t(4096));
  g.M = M; g.N = N; g.K = K; g.ta = ta; g.tb = tb; g.epi = Epi(epi); g.c_f32 = c_f32;
  g.lda = ta ? M : K; g.ldb = tb ? K : N; g.ldc = N;
  if (ws_floats) { g.ws = reinterpret_cast<float*>(uintptr_t(4096)); g.ws_floats = size_t(ws_floats); }
  return g;
}
extern "C" int path(int dt, int M, int N, int K, int ta, int tb, int epi, int c_f32) {
  return gemm_path(dt, make(M, N, K, ta, tb, epi, c_f32, 0));
}
extern "C" int dma_variant(int M, int N, int K, int tb) { return gemm_dma_variant(make(M, N, K, 0, tb, EPI_STORE, 0, 0)); }
// a forward product whose first operand's rows are lda elements apart: path, variant, whether the lean k loop takes it
extern "C" int far_rows(int M, int N, int K, long long lda) {
  Gemm g = make(M, N, K, 0, 0, EPI_BIAS, 1, 0);
  g.lda = lda;
  return gemm_path(1, g) * 100 + gemm_dma_variant(g) * 10 + gemm_lean_ok(g);
}
// the tile of a weight gradient over the same rows
extern "C" int far_wgrad(int M, int N, int K, long long lda) {
  Gemm g = make(M, N, K, 1, 0, EPI_STORE, 1, 1 << 24);
  g.lda = lda;
  return wgrad_tiling(&g, 1).tile * 10 + gemm_lean_ok(g);
}
// a block's four weight gradients with the workspace that the plan gives them at least
extern "C" int block_wgrads(int D, int F, int tokens) {
  const size_t ws = gemm_wgrad_batch_ws_floats(D, F);
  const Gemm g[4] = {make(F, D, tokens, 1, 0, EPI_STORE, 1, ws), make(D, F, tokens, 1, 0, EPI_STORE, 1, ws),
                     make(D, D, tokens, 1, 0, EPI_STORE, 1, ws), make(D, 3 * D, tokens, 1, 0, EPI_STORE, 1, ws)};
  const WgradTiling t = wgrad_tiling(g, 4);
  return t.tile * 100 + t.splits;
}
extern "C" int f32_tile(int M, int N, int K, int ta, int tb) {
  const Gemm g = make(M, N, K, ta, tb, EPI_STORE, 1, 0);
  const F32Tile t = gemm_f32_tile(&g, 1);
  return t.tm * 10 + t.tn;
}
// the same in the kernel that stages its tiles through registers
extern "C" int f32_staged_tile(int M, int N, int K, int ta, int tb) {
  const Gemm g = make(M, N, K, ta, tb, EPI_STORE, 1, 0);
  const F32Tile t = gemm_f32_tile(&g, 1, false);
  return t.tm * 10 + t.tn;
}
extern "C" int f32_block_wgrads(int D, int F, int tokens) {
  const Gemm g[4] = {make(F, D, tokens, 1, 0, EPI_STORE, 1, 0), make(D, F, tokens, 1, 0, EPI_STORE, 1, 0),
                     make(D, D, tokens, 1, 0, EPI_STORE, 1, 0), make(D, 3 * D, tokens, 1, 0, EPI_STORE, 1, 0)};
  const F32Tile t = gemm_f32_tile(g, 4);
  return t.tm * 10 + t.tn;
}
extern "C" int reg_tiling(int M, int N, int K, int ta, int epi, int c_f32, long long ws_floats) {
  const GemmRegTiling t = gemm_reg_tiling(make(M, N, K, ta, 0, epi, c_f32, ws_floats));
  return t.tile * 100 + t.splits;
}
"""

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            so = os.path.join(d, "rules.so")
            subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-x", "c++", "-", "-o", so],
                           input=SOURCE.encode(), check=True)
            _lib = ctypes.CDLL(so)
        _lib.far_rows.argtypes = _lib.far_wgrad.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong]
        _lib.reg_tiling.argtypes = [ctypes.c_int] * 6 + [ctypes.c_longlong]
    return _lib


def forward(tokens, K, N, epi, c_f32=False, dt=1):
    return lib().path(dt, tokens, N, K, 0, 0, epi, int(c_f32))


def input_gradient(tokens, K, N, epi=STORE, c_f32=False, dt=1):
    return lib().path(dt, tokens, N, K, 0, 1, epi, int(c_f32))


def weight_gradient(rows, cols, tokens, dt=1):
    return lib().path(dt, rows, cols, tokens, 1, 0, STORE, 1)


# variants of the asynchronous kernels
T128, T256x128, T64, T128_EIGHT_WAVES, TWO_GROUPS_256, TWO_GROUPS_192, T128x64 = 1, 2, 3, 4, 5, 6, 7


def dma_variant(M, N, K, tb=False):
    """tiles of a forward (tb: input-gradient) product"""
    return lib().dma_variant(M, N, K, int(tb))


def far_rows(M, N, K, lda):
    """(path, variant, lean) of a forward product over rows lda elements apart"""
    r = lib().far_rows(M, N, K, lda)
    return r // 100, r // 10 % 10, bool(r % 10)


def far_wgrad(M, N, K, lda):
    """(tile, lean) of a weight gradient over rows lda elements apart"""
    r = lib().far_wgrad(M, N, K, lda)
    return r // 10, bool(r % 10)


def reg_tiling(M, N, K, ta, epi=STORE, c_f32=False, ws_floats=0):
    """(tile, splits) of the register-staged kernel"""
    t = lib().reg_tiling(M, N, K, int(ta), epi, int(c_f32), ws_floats)
    return t // 100, t % 100


def block_wgrads(D, F, tokens):
    """(tile, splits) of a block's four weight gradients in bf16 mode"""
    t = lib().block_wgrads(D, F, tokens)
    return t // 100, t % 100


def f32_tile(M, N, K, tb=False):
    """tile of an fp32 forward (tb: input-gradient) product, in units of 32"""
    return divmod(lib().f32_tile(M, N, K, 0, int(tb)), 10)


def f32_staged_tile(M, N, K, ta=False, tb=False):
    """the same for rows that are no 16-byte pieces"""
    return divmod(lib().f32_staged_tile(M, N, K, int(ta), int(tb)), 10)


def f32_block_wgrads(D, F, tokens):
    return divmod(lib().f32_block_wgrads(D, F, tokens), 10)
