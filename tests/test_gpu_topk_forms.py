"""The forms of the top-K baseline's two small kernels, at the edges of their ranges: rows of 1, 64, 65, 256, 257 and 513 chunks of 16 bytes for the
draft logits, 255 to 513 vocabulary tiles for the tail."""
import pytest

import workloads as wl
from parity import make_inputs
from test_gpu_topk import check, planted_drafts, run_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [1, 64, 65, 256, 257, 513])
@pytest.mark.parametrize("base,per", [("8b_b1_k16", 8), ("tiny_f32", 4)])
def test_draft_logits(base, per, chunks):
    w = wl.scaled(wl.WORKLOADS[base], name="topk_rows", B=2, K=5, d_t=chunks * per, d_d=0, V=601)
    x = make_inputs(w, 41)
    draft = planted_drafts(x, 41)
    out, _ = run_topk(x, draft, (2,))
    check(x, draft, out[2], 2)


@pytest.mark.parametrize("V", [255 * 128, 256 * 128, 256 * 128 + 1, 512 * 128, 512 * 128 + 1])
def test_tail_tiles(V):
    import paper_2504_20039_amd as aj
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="topk_tiles", B=2, K=3, d_t=72, d_d=0, V=V)
    x = make_inputs(w, 42)
    draft = planted_drafts(x, 42)
    draft[0, 0] = V - 1                                  # an entry of the last tile
    out, name = run_topk(x, draft, (2,), aj.AJ_KERNEL_TILE)
    assert name == "lm_head_tile_bf16"                   # tiles of 128 vocabulary rows
    check(x, draft, out[2], 2)
