"""The attention kernels on the fp32 matrix instructions at the edges of their tiles: sequences that end on, before and
behind a 16-row fragment or a 64-row tile, head sizes that fill a column block (16, 32, 64, 128) or leave columns of it
empty.  fp32 mode against the exact oracle at 1e-4, as for every other shape; bf16 with head sizes other than 64 takes
the same kernels (tests/test_gpu_small_shapes.py)."""
import pytest

from paper_2102_03161_amd import binding
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu

# (tokens, heads, head size)
CASES = [(16, 2, 16), (17, 3, 8), (63, 2, 32), (64, 2, 64), (65, 2, 128), (80, 2, 24), (129, 2, 40), (197, 3, 64), (257, 2, 104),
         (1216, 2, 8), (832, 1, 128)]   # the longest sequences of these head sizes


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


@pytest.mark.parametrize("S,heads,dh", CASES)
def test_fp32_attention_at_tile_edges(torch_mod, S, heads, dh):
    print(f"fp32 attention S={S} heads={heads} dh={dh}", flush=True)
    w = dict(arch="bert", L=2, D=heads * dh, H=heads, F=64, S=S, n_out=2, img=0, patch=0, chans=0, vocab=50, max_pos=S,
             ln_eps=1e-12, B=2, optimizer="adamw", dtype="f32")
    ctx = binding.Context(binding.make_config(w))
    vals = H.init_values(w, ctx, 7)
    H.load_params(ctx, vals)
    x, y = H.batch_for(w, 7, 2)
    g = H.gpu_step(torch_mod, ctx, w, x, y, 0)
    ctx.close()
    o = H.oracle_step(w, vals, x, y, 0)
    H.oracle_update(w, o, vals, g["grads"], 0)
    H.compare_step(w, g, o, 0, 1e-4, rss=H.summand_rss(w, vals, x, y, 0))
