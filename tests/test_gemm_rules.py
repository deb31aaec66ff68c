"""Which kernel the products of the training step take, without a GPU."""
import pytest

from tests import gemm_rules as R
from tests import test_gpu_gemm_tiles as G
from tests.test_gpu_parity import MANY_TOKENS
from tests.test_gpu_wgrad_riders import CASE as RIDERS


@pytest.mark.parametrize("tokens", [1, 24, 200, 4096, 12288])
@pytest.mark.parametrize("F", [100, 1028, 3076, 4300])
def test_mlp_widths_that_are_no_multiple_of_8_stay_on_the_bf16_matrix_instructions(tokens, F):
    """F % 4 == 0 is accepted: the first MLP product (for any number of rows: a row's result must not depend on the
    batch) and both MLP weight gradients have a strided operand of that width."""
    D = 768
    assert R.forward(tokens, D, F, R.BIAS_GELU) == R.REG
    few = tokens <= 32                                   # nothing but the write of the result
    assert R.weight_gradient(D, F, tokens) == (R.F32 if few else R.REG)      # W1
    assert R.weight_gradient(F, D, tokens) == (R.F32 if few else R.REG)      # W2
    assert R.input_gradient(tokens, D, F, R.MUL_DGELU) == R.DMA
    # k-major operands of that width have no 16-byte pieces
    assert R.forward(tokens, F, D, R.BIAS_RES) == R.F32
    assert R.input_gradient(tokens, F, D) == R.F32


def test_patch_and_class_counts_that_are_no_multiple_of_8():
    assert R.weight_gradient(588, 768, 64 * 256) == R.REG             # 14 x 14 x 3 patches
    assert R.forward(64, 768, 100, R.BIAS, c_f32=True) == R.REG       # 100 classes
    assert R.weight_gradient(768, 100, 64) == R.REG
    assert R.weight_gradient(768, 10, 64) == R.F32                    # fewer than 32 columns
    assert R.forward(64, 768, 10, R.BIAS, c_f32=True) == R.F32
    assert R.forward(64, 768, 101, R.BIAS, c_f32=True) == R.F32       # odd


def test_multiples_of_8_take_the_asynchronous_kernels():
    for tokens in (1, 231, 12608):
        assert R.forward(tokens, 768, 3072, R.BIAS_GELU) == R.DMA
        assert R.input_gradient(tokens, 3072, 768) == R.DMA
        assert R.weight_gradient(768, 3072, tokens) == R.DMA
        assert R.forward(tokens, 768, 3072, R.BIAS_GELU, dt=0) == R.F32


def test_contractions_that_are_no_multiple_of_64():
    """Many rows take 128x128 tiles, whatever K; few rows 64x64."""
    for tb in (False, True):
        for M, N, K in [(16384, 1152, 4304), (32768, 600, 200), (16384, 984, 328), (8192, 3072, 776), (4096, 800, 200)]:
            assert R.dma_variant(M, N, K, tb) == R.T128_EIGHT_WAVES, (M, N, K)
        for M, N, K in [(4096, 768, 3104), (16384, 768, 800)]:
            assert R.dma_variant(M, N, K, tb) == R.T128, (M, N, K)
        for M, N, K in [(1024, 1152, 4304), (200, 768, 3080), (4096, 200, 200), (2639, 768, 3104), (4096, 480, 160)]:
            assert R.dma_variant(M, N, K, tb) == R.T64, (M, N, K)


def test_variants_take_the_contractions_they_are_given():
    for M in (1, 7, 64, 500, 1379, 4096, 5000, 8192, 12608, 25216, 32768):
        for N in (8, 200, 768, 1152, 2304, 3072, 4096):
            for K in range(8, 4400, 8):
                for tb in (False, True):
                    v = R.dma_variant(M, N, K, tb)
                    need = {R.T128: 32, R.T256x128: 32, R.TWO_GROUPS_256: 64, R.TWO_GROUPS_192: 64, R.T128x64: 64}.get(v, 8)
                    assert K % need == 0, (M, N, K, tb, v)


# us of each variant on a MI355X, weights from HBM: (rows, columns, contraction, input gradient)
MEASURED = {
    (520, 1024, 4096, False): {3: 20.2, 7: 26.8, 1: 47.4, 4: 54.6},
    (1379, 768, 3072, False): {3: 21.6, 7: 22.4, 1: 38.6, 4: 41.9},
    (1379, 3072, 768, False): {3: 18.5, 7: 19.8, 1: 20.6, 4: 20.2},
    (2000, 3072, 1024, False): {3: 24.7, 7: 21.5, 1: 21.5, 4: 22.6},
    (2639, 768, 768, False): {3: 9.4, 7: 8.5, 1: 12.9, 4: 13.7},
    (2900, 768, 3072, False): {3: 34.0, 7: 31.1, 1: 39.1, 4: 42.5},
    (3300, 768, 768, False): {3: 12.0, 7: 11.2, 1: 13.5, 4: 13.9},
    (3152, 1024, 4096, False): {3: 56.6, 7: 43.4, 1: 58.7, 4: 63.0},
    (3152, 1024, 3072, True): {3: 44.7, 7: 34.3, 1: 44.8, 4: 47.6},
    (4000, 768, 3072, False): {3: 36.5, 7: 31.9, 1: 40.7, 4: 43.4},
    (4000, 768, 3072, True): {3: 36.5, 7: 33.2, 1: 43.1, 4: 46.4},
    (4096, 768, 3072, False): {3: 37.1, 7: 33.2, 1: 43.1, 4: 43.4, 5: 65.6, 6: 56.4},
    (4400, 768, 2304, True): {3: 34.2, 7: 27.6, 1: 35.7, 4: 37.0, 5: 55.8, 6: 47.2},
    (4600, 512, 2048, False): {3: 23.6, 7: 21.8, 1: 29.2, 4: 30.9, 5: 47.7, 6: 40.9},
    (6500, 384, 1536, False): {3: 18.5, 7: 17.4, 1: 22.1, 4: 23.4, 5: 36.8, 6: 32.1},
    (8192, 1536, 384, False): {3: 27.6, 7: 25.8, 1: 25.2, 4: 24.4, 5: 28.2, 6: 38.9},
    (8192, 768, 3072, True): {3: 70.9, 7: 61.9, 1: 64.0, 4: 59.0, 5: 78.1, 6: 65.2},
    (8192, 3072, 768, True): {3: 74.8, 7: 65.6, 1: 62.8, 4: 53.9, 2: 57.0, 5: 60.4, 6: 67.3},
    (12608, 768, 3072, False): {3: 109.6, 7: 91.0, 1: 89.4, 4: 91.0, 5: 78.4, 6: 68.1},
    (12608, 2304, 768, False): {3: 83.4, 7: 72.4, 1: 63.2, 4: 61.7, 5: 53.2, 6: 62.2},
}


@pytest.mark.parametrize("shape", MEASURED)
def test_tiles_are_near_the_fastest_measured(shape):
    us = MEASURED[shape]
    assert us[R.dma_variant(*shape)] <= 1.05 * min(us.values())


@pytest.mark.parametrize("S,D", [(512, 1024), (4096, 2048), (8192, 1024), (8192, 2048), (16384, 2048), (32768, 2048)])
@pytest.mark.parametrize("rows", [1, 4, 64, 100, 128, 512])
def test_rows_far_apart_stay_on_the_asynchronous_kernels(rows, S, D):
    """The head's products over first tokens: rows S * D elements apart.  A lane's offsets within a tile are 32 bits wide
    in the kernels of 64-column tiles and small weight gradients, which take what fits and no more."""
    lda = S * D
    path, variant, lean = R.far_rows(rows, 8, D, lda)
    assert path == R.DMA
    assert lean == ((min(rows, 128) - 1) * lda * 2 + 256 < 2 ** 32)
    assert lean or variant not in (R.T64, R.T128x64)
    tile, lean = R.far_wgrad(D, 8, rows, lda)
    assert lean == (63 * lda * 2 + 256 < 2 ** 32)
    assert lean or tile == 256


@pytest.mark.parametrize("name", G.CASES)
def test_gpu_cases_take_the_kernels_they_are_there_for(name):
    G.takes_its_kernels(name)


def test_other_gpu_tests_take_the_weight_gradients_they_are_there_for():
    w = RIDERS[0]
    assert R.block_wgrads(w["D"], w["F"], w["B"] * w["S"]) == (256, 3)
    for D, (B, wgrads, tiles) in MANY_TOKENS.items():
        assert R.block_wgrads(D, 1728, 65 * B) == wgrads and R.dma_variant(65 * B, 1728, D) == tiles
    assert R.block_wgrads(768, 3072, 64 * 197) == (256, 2)


# us of 32x32, 32x64, 64x64 and 128x128 tiles on a MI355X, staged through registers: (rows, columns, contraction)
MEASURED_STAGED = {
    (197, 768, 147): (5.6, 7.6, 10.7, 26.3),
    (800, 768, 147): (8.8, 9.7, 11.0, 26.6),
    (1568, 1024, 363): (36.4, 32.0, 29.1, 49.0),
    (2500, 256, 49): (5.4, 6.3, 7.2, 17.2),
    (6400, 256, 363): (36.7, 32.2, 29.1, 48.6),
    (8192, 1024, 147): (62.0, 52.7, 47.2, 44.1),
    (12544, 256, 363): (59.4, 52.1, 51.4, 50.1),
}


@pytest.mark.parametrize("shape", MEASURED_STAGED)
def test_fp32_staged_tiles_are_near_the_fastest_measured(shape):
    us = dict(zip([(1, 1), (1, 2), (2, 2), (4, 4)], MEASURED_STAGED[shape]))
    assert us[R.f32_staged_tile(*shape)] <= 1.05 * min(us.values())


def test_fp32_tiles():
    rows = {50: (1, 1), 450: (1, 2), 2000: (2, 2), 4081: (4, 4)}
    assert {m: R.f32_tile(m, 1024, 768) for m in rows} == rows
    assert R.f32_tile(1576, 768, 3072) == R.f32_tile(1576, 768, 2304, tb=True) == (2, 3)


def test_weight_gradients_are_not_cut_finer_than_their_k_tiles():
    for D, F in [(64, 256), (200, 800), (256, 1024), (384, 1536), (512, 2048), (768, 3072), (1024, 4096), (2048, 8192)]:
        for tokens in list(range(1, 600, 7)) + list(range(600, 40000, 131)):
            tile, splits = R.block_wgrads(D, F, tokens)
            nk = -(-tokens // 64)
            assert tile in (64, 128, 256) and 1 <= splits <= 16 and splits <= nk, (D, F, tokens)
