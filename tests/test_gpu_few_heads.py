"""Attention backward on one or two workgroups per head (up to half as many heads as CUs: two), at the edges of the rule and
of the 32-row tiles, and the LayerNorm backward's workgroup sums at widths of up to eight vectors per lane.  bf16 mode against
the exact oracle (or the bf16 storage model) at 2e-2, value by value; fp32 mode at 1e-4."""
import pytest

from tests.test_gpu_gemm_tiles import BERT, VIT, check_fp32_step, check_step, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,heads,B", [(33, 4, 32), (33, 4, 33), (64, 2, 3), (97, 2, 1), (129, 1, 2), (203, 3, 2), (256, 2, 1)])
def test_backward_with_few_heads(torch_mod, S, heads, B):  # noqa: F811
    """128 heads take two workgroups each on 256 CUs, 132 heads one; one to eight tiles of 32 rows, full and ragged."""
    w = dict(BERT, L=2, D=64 * heads, H=heads, F=256, S=S, max_pos=S, B=B)
    check_step(torch_mod, f"{B * heads} heads of {S} tokens", w, 0, B, 60 + S)


@pytest.mark.parametrize("D,dtype", [(8, "f32"), (256, "f32"), (1280, "f32"), (1280, "bf16"), (2048, "bf16")])
def test_layernorm_backward_sums(torch_mod, D, dtype):  # noqa: F811
    """7 x 17 rows: the last workgroup's waves have no row."""
    w = dict(VIT, L=1, D=D, H=max(1, D // 64), F=4 * 64, img=32, S=17, n_out=10, B=7, dtype=dtype)
    if dtype == "f32":
        check_fp32_step(torch_mod, w, 71)
    else:
        check_step(torch_mod, f"width {D}", w, 0, 7, 72)
