"""Shapes at which the matrix-core products change kernel: fewer rows than a tile, token counts that are no multiple of a
k tile, 64- and 128-wide tiles, split and unsplit weight gradients, the eight-wave tiles of the input gradients.  bf16
mode against the exact oracle (or the bf16 storage model) at 2e-2, value by value; and rows of the frozen prefix bit by
bit between batches whose products run on different tiles."""
import numpy as np
import pytest

from paper_2102_03161_amd import binding
from tests import gemm_rules as R
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

VIT = dict(arch="vit", img=56, patch=8, chans=3, S=50, vocab=0, max_pos=0, ln_eps=1e-6, optimizer="adamw", dtype="bf16")
BERT = dict(arch="bert", img=0, patch=0, chans=0, n_out=2, vocab=500, ln_eps=1e-12, optimizer="adamw", dtype="bf16")

CASES = {
    # one sample: 50 tokens, products of a single row, a contraction over 1000 classes
    "one_row": (dict(VIT, L=2, D=256, H=4, F=1024, n_out=1000, B=1), 0, 1, 41),
    # 350 tokens at full width: 64-row tiles, 128-wide weight gradients over five and a half k tiles, seven-row products
    # with a split contraction
    "few_rows": (dict(VIT, L=2, D=768, H=12, F=3072, n_out=1000, B=7), 0, 7, 42),
    # 2156 tokens, narrow matrices: 64-wide weight-gradient tiles, the contraction in four parts
    "narrow_split": (dict(BERT, L=2, D=256, H=4, F=1024, S=77, max_pos=80, B=28), 0, 28, 43),
    # 7161 tokens of width 384: 128-wide ones in four parts
    "medium_split": (dict(BERT, L=1, D=384, H=6, F=1536, S=77, max_pos=80, B=93), 0, 93, 50),
    # 4851 tokens: the two-group weight-gradient kernel with a partial last k tile, in five parts, whose slabs the next
    # block's launch adds
    "group_tail": (dict(BERT, L=2, D=512, H=8, F=2048, S=77, max_pos=80, B=63), 0, 63, 44),
    # 3850 x 800 x 200: 128x128 tiles of eight waves with an eighth of a k tile at the end, forward and backward
    "eight_waves_tail": (dict(BERT, L=1, D=200, H=25, F=800, S=77, max_pos=80, B=50), 0, 50, 49),
    # 2639 x 3072 input gradients: 504 tiles of 128x128, eight waves each
    "eight_waves": (dict(BERT, L=1, D=768, H=12, F=3072, S=203, max_pos=203, B=13), 0, 13, 45),
}

# what the cases above are there for: the tile and the parts of a block's weight gradients ...
BLOCK_WGRADS = {"few_rows": (128, 1), "narrow_split": (64, 4), "medium_split": (128, 4), "group_tail": (256, 5)}
# ... and the tiles of an input gradient, (rows, columns, contraction)
INPUT_GRADIENT = {"few_rows": ((350, 768, 3072), R.T64), "eight_waves": ((2639, 3072, 768), R.T128_EIGHT_WAVES),
                  "eight_waves_tail": ((3850, 800, 200), R.T128_EIGHT_WAVES)}


def takes_its_kernels(name):
    w, _, nb, _ = CASES[name]
    if name in BLOCK_WGRADS:
        assert R.block_wgrads(w["D"], w["F"], nb * w["S"]) == BLOCK_WGRADS[name]
    if name in INPUT_GRADIENT:
        (M, N, K), variant = INPUT_GRADIENT[name]
        assert R.dma_variant(M, N, K, tb=True) == variant


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


def check_step(torch, name, w, k, nb, seed):
    print(f"tile edges: {name}", flush=True)
    ctx = binding.Context(binding.make_config(w, B=nb))
    vals = H.init_values(w, ctx, seed)
    H.load_params(ctx, vals)
    x, y = H.batch_for(w, seed, nb)
    g = H.gpu_step(torch, ctx, w, x, y, k)
    ctx.close()
    o = H.oracle_step(w, vals, x, y, k)
    m = H.storage_model_step(w, vals, x, y, k)
    H.compare_step(w, g, o, k, 2e-2, check_params=False, model=m, rss=H.summand_rss(w, vals, x, y, k))


def prefix_rows(torch, w):
    ctx = binding.Context(binding.make_config(w))
    H.load_params(ctx, H.init_values(w, ctx, 5))
    ctx.set_freeze_boundary(2)
    x = H.to_dev(torch, H.batch_for(w, 5, 65)[0])
    rows = {}
    for nb in (65, 7, 1):
        ctx.frozen_forward(x[:nb].contiguous())
        rows[nb] = ctx.read_activation(binding.ACT_HK, (nb, w["S"], w["D"]))
    ctx.close()
    for nb in (7, 1):
        assert np.array_equal(rows[nb], rows[65][:nb]), nb


@pytest.mark.parametrize("name", CASES)
def test_products_at_tile_edges(torch_mod, name):
    w, k, nb, seed = CASES[name]
    takes_its_kernels(name)
    check_step(torch_mod, name, w, k, nb, seed)


# 64-column tiles: (rows, columns, contraction) of an input gradient and its tiles
NARROW_CASES = {
    # 128x64 tiles with 79 rows in the last one; 128-wide weight-gradient tiles with a partial k tile
    "narrow": (dict(BERT, L=1, D=768, H=12, F=3072, S=203, max_pos=203, B=13), 51, (2639, 768, 3072), R.T128x64),
    # 64x64 tiles, one to a CU, four stages: 520 = 8 k tiles and an eighth
    "four_stages_tail": (dict(BERT, L=2, D=256, H=4, F=520, S=77, max_pos=80, B=6), 52, (462, 256, 520), R.T64),
    # three stages: 392 = 6 k tiles and an eighth
    "three_stages_tail": (dict(BERT, L=2, D=256, H=4, F=392, S=77, max_pos=80, B=6), 53, (462, 256, 392), R.T64),
}


@pytest.mark.parametrize("name", NARROW_CASES)
def test_64_column_tiles(torch_mod, name):
    w, seed, (M, N, K), variant = NARROW_CASES[name]
    assert w["B"] * w["S"] == M and R.dma_variant(M, N, K, tb=True) == variant
    check_step(torch_mod, name, w, 0, w["B"], seed)


def test_prefix_rows_do_not_depend_on_128x64_tiles(torch_mod):
    """3250 rows of width 1024 take 128x64 tiles in the second MLP product, 350 and 50 rows 64x64 ones."""
    assert [R.dma_variant(50 * nb, 1024, 4096) for nb in (65, 7, 1)] == [R.T128x64, R.T64, R.T64]
    prefix_rows(torch_mod, dict(VIT, L=2, D=1024, H=16, F=4096, n_out=10, B=65))


# rows that are even but no multiple of 8 elements long
EVEN_CASES = {
    # patches of 588 values, 1028-wide MLP, 100 classes: register-staged 64x64 tiles, split contractions with a k tail
    "patch14": (dict(VIT, img=56, patch=14, S=17, L=2, D=256, H=4, F=1028, n_out=100, B=33), 0, 33, 46),
    # the same on 17 rows, the patch weights frozen
    "patch14_few_rows": (dict(VIT, img=56, patch=14, S=17, L=2, D=256, H=4, F=1028, n_out=102, B=1), 1, 1, 47),
    # 2926 tokens: 128x128 tiles in the forward product and (split) in both MLP weight gradients
    "mlp3076": (dict(BERT, L=1, D=768, H=12, F=3076, S=77, max_pos=80, B=38), 0, 38, 48),
}


@pytest.mark.parametrize("name", EVEN_CASES)
def test_rows_that_are_no_multiple_of_8_long(torch_mod, name):
    w, k, nb, seed = EVEN_CASES[name]
    tokens, D, F = nb * w["S"], w["D"], w["F"]
    assert R.forward(tokens, D, F, R.BIAS_GELU) == R.REG
    assert R.weight_gradient(D, F, tokens) == R.weight_gradient(F, D, tokens) == (R.REG if tokens > 32 else R.F32)
    check_step(torch_mod, name, w, k, nb, seed)


def test_even_rows_of_the_prefix_do_not_depend_on_the_tiles(torch_mod):
    """MLP width 3076: the first product on 128x128 and 64x64 register-staged tiles, the second on 64x64 and 32x32 tiles of
    the fp32 instructions."""
    assert [R.reg_tiling(50 * nb, 3076, 768, False, R.BIAS_GELU)[0] for nb in (65, 7, 1)] == [128, 64, 64]
    prefix_rows(torch_mod, dict(VIT, L=2, D=768, H=12, F=3076, n_out=10, B=65))


def test_prefix_rows_with_a_k_tail_do_not_depend_on_the_tiles(torch_mod):
    """Width 200, MLP width 1000: the first MLP product on 128x128 tiles of eight waves and on 64x64 tiles, both with a
    partial last k tile."""
    assert [R.dma_variant(50 * nb, 1000, 200) for nb in (65, 7, 1)] == [R.T128_EIGHT_WAVES, R.T64, R.T64]
    prefix_rows(torch_mod, dict(VIT, L=2, D=200, H=25, F=1000, n_out=10, B=65))


def check_fp32_step(torch, w, seed):
    ctx = binding.Context(binding.make_config(w))
    vals = H.init_values(w, ctx, seed)
    H.load_params(ctx, vals)
    x, y = H.batch_for(w, seed, w["B"])
    g = H.gpu_step(torch, ctx, w, x, y, 0)
    ctx.close()
    o = H.oracle_step(w, vals, x, y, 0)
    H.oracle_update(w, o, vals, g["grads"], 0)
    H.compare_step(w, g, o, 0, 1e-4, rss=H.summand_rss(w, vals, x, y, 0))


# tiles of a block's forward products and input gradients of 50 rows per sample, and of its weight gradients
FP32_EDGES = {(1, 3072): ({(1, 1)}, (1, 1)), (9, 3072): ({(1, 1), (1, 2), (2, 3)}, (2, 2)), (40, 3072): ({(2, 2), (2, 3)}, (2, 2)),
              (3, 1028): ({(1, 1), (1, 2)}, (2, 2))}


@pytest.mark.parametrize("nb,F", FP32_EDGES)
def test_fp32_products_at_tile_edges(torch_mod, nb, F):
    """fp32 mode: 50, 450 and 2000 rows of width 768 and MLP width 3072 take 32x32 tiles, these with 32x64 and 64x96 ones, and
    64x64 and 64x96 ones, their weight gradients 32x32 and 64x64; ten classes take the register-staged loads, a width of 1028
    the ragged edges."""
    print(f"fp32 tile edges: nb={nb} F={F}", flush=True)
    D, rows = 768, 50 * nb
    forward = {R.f32_tile(rows, N, K) for N, K in [(3 * D, D), (D, D), (F, D), (D, F)]}
    backward = {R.f32_tile(rows, N, K, tb=True) for N, K in [(D, 3 * D), (D, D), (D, F), (F, D)]}
    assert (forward | backward, R.f32_block_wgrads(D, F, rows)) == FP32_EDGES[nb, F]
    check_fp32_step(torch_mod, dict(VIT, L=2, D=768, H=12, F=F, n_out=10, B=nb, dtype="f32"), 6)


@pytest.mark.parametrize("S,nb", [(203, 1), (77, 7)])
def test_fp32_weight_gradients_on_the_largest_tiles(torch_mod, S, nb):
    """fp32 mode, width 1024: a block's weight gradients on 128x128 tiles over six k tiles and 11 tokens, sixteen and 27."""
    assert R.f32_block_wgrads(1024, 4096, S * nb) == (4, 4)
    print(f"fp32 weight gradients of width 1024 over {S * nb} tokens", flush=True)
    check_fp32_step(torch_mod, dict(BERT, L=1, D=1024, H=16, F=4096, S=S, max_pos=203, B=nb, dtype="f32"), 11)


def test_fp32_products_on_the_largest_tiles(torch_mod):
    """fp32 mode: 4081 x 1024 forward products and input gradients are 256 tiles of 128x128."""
    assert R.f32_tile(4081, 1024, 256) == R.f32_tile(4081, 1024, 256, tb=True) == (4, 4)
    check_fp32_step(torch_mod, dict(BERT, L=1, D=256, H=4, F=1024, S=77, max_pos=80, B=53, dtype="f32"), 8)


# samples of 64 patches of 147 values, width 512: tiles of the patch embedding, staged through registers
STAGED = {3: (1, 1), 31: (1, 2), 51: (2, 2), 255: (4, 4)}


@pytest.mark.parametrize("nb", STAGED)
def test_fp32_tiles_staged_through_registers(torch_mod, nb):
    """fp32 mode: an odd contraction, forward and (rows of 147) in the weight gradient, on each tile size."""
    assert R.f32_staged_tile(64 * nb, 512, 147) == STAGED[nb]
    print(f"fp32 staged tiles: nb={nb}", flush=True)
    check_fp32_step(torch_mod, dict(VIT, patch=7, S=65, L=1, D=512, H=8, F=64, n_out=10, B=nb, dtype="f32"), 10)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_prefix_rows_do_not_depend_on_the_tiles(torch_mod, dtype):
    """3250 rows take 128x128 tiles in the wide products, 50 and 350 rows smaller ones."""
    prefix_rows(torch_mod, dict(VIT, L=2, D=768, H=12, F=3072, n_out=10, B=65, dtype=dtype))


def test_fp32_bias_gradients_over_many_tokens(torch_mod):
    """fp32 mode: the patch bias gradient is the sum of the patch rows' gradients over 12544 tokens, the position
    gradients are the same rows summed over 49 samples each.  Their sum in 64 bits is the reference: its own error,
    chains of 49 rows averaged over 256 positions, is about 1e-8.  These rows mostly agree in sign (their sum is 16 times
    its root-sum-square); on such columns the kernel's order of additions is 5e-8 off, one chain over all tokens
    1.7e-6 (both emulated on N(1, 1)).  The bar is 4 times the former."""
    w = dict(VIT, L=2, D=64, H=4, F=256, img=64, patch=4, S=257, n_out=10, B=49, dtype="f32")
    ctx = binding.Context(binding.make_config(w))
    H.load_params(ctx, H.init_values(w, ctx, 9))
    x, y = H.batch_for(w, 9, 49)
    grads = H.gpu_step(torch_mod, ctx, w, x, y, 0)["grads"]
    ctx.close()
    want = grads["front.pos"].astype(np.float64)[1:].sum(0)
    err = np.linalg.norm(grads["front.b_pe"].ravel() - want) / np.linalg.norm(want)
    print(f"patch bias gradient over 12544 tokens: {err:.2e}", flush=True)
    assert err < 2e-7
