"""The small-tile kernel at the edges of its tiles: 1 to 4 vocabulary blocks per wave, every kind of row tile, hidden sizes that
end inside a line and inside a slab, odd and even numbers of slabs, through every entry point's epilogue."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import check_small_tile, compare, make_inputs, run_gpu
from test_gpu_parity import oracle_greedy
import test_gpu_topk as tk

pytestmark = pytest.mark.gpu


def logit_bound(w, x):
    # products of bf16 values are exact in fp32; |fp32 sum of d products - exact| <= d 2^-24 sum |a b| in any order
    return (w.d_t + 1) * 2.0**-24 * np.linalg.norm(wl.widen(x.ht).astype(np.float64), axis=1)[:, None] * \
        np.linalg.norm(wl.widen(x.W).astype(np.float64), axis=1)[None, :]


def check_logits(w, x, tile, wdev, *w_dtype):
    import torch
    import paper_2504_20039_amd as aj
    h = aj.aj_create(w.B, w.K, w.d_t, w.d_d, w.V, aj.AJ_BF16, 1, 0, 0, *w_dtype)
    check_small_tile(h, *tile)
    logits = torch.empty((w.M, w.V), dtype=torch.float32, device="cuda")
    aj.aj_debug_logits(h, aj.device_tensor(x.ht), aj.device_tensor(wdev), logits)
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    ref = wl.widen(x.ht).astype(np.float64) @ wl.widen(x.W).astype(np.float64).T
    assert (np.abs(logits.cpu().numpy() - ref) <= logit_bound(w, x)).all()


@pytest.mark.parametrize("tile,shape", [               # tile: vocabulary blocks of 64, verify-row blocks of 16, waves
    ((1, 1, 4), dict(B=1, K=1, d_t=8, d_d=0, V=12289)),             # one ragged slab; tiles of 52 vocabulary rows, a last one of 17
    ((1, 1, 4), dict(B=1, K=9, d_t=264, d_d=8, V=12352)),           # two slabs, the second of 8 elements
    ((1, 4, 4), dict(B=3, K=20, d_t=1000, d_d=64, V=12300)),        # 52-row tiles, four row blocks
    ((2, 3, 8), dict(B=1, K=32, d_t=512, d_d=64, V=16389)),         # four slabs
    ((2, 8, 8), dict(B=4, K=29, d_t=384 * 2, d_d=64, V=20001)),
    ((3, 3, 12), dict(B=3, K=15, d_t=96, d_d=0, V=33001)),           # two slabs, the second half empty
    ((3, 7, 12), dict(B=5, K=39, d_t=320, d_d=64, V=16400)),         # 200 rows: two row tiles, an odd number of slabs
    ((3, 6, 12), dict(B=9, K=28, d_t=256, d_d=64, V=14000)),         # 261 rows: three row tiles
    ((3, 3, 12), dict(B=1, K=47, d_t=160, d_d=0, V=33025)),          # a last tile of 25 vocabulary rows
    ((3, 8, 12), dict(B=4, K=29, d_t=256, d_d=64, V=40001)),
    ((3, 7, 12), dict(B=2, K=149, d_t=328, d_d=0, V=12500)),         # 300 rows: three row tiles, the last one short
    ((4, 1, 16), dict(B=1, K=11, d_t=72, d_d=0, V=50177)),           # a last tile of 49 vocabulary rows
    ((4, 4, 16), dict(B=3, K=20, d_t=136, d_d=8, V=50257)),
    ((4, 6, 8), dict(B=3, K=30, d_t=328, d_d=64, V=50001)),
])
def test_bf16_shapes(tile, shape):
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="slab", p_match=0.6, **shape)
    x = make_inputs(w, 3)
    greedy = oracle_greedy(x)
    draft = wl.draft_tokens(w, 3, greedy[0])
    gpu = run_gpu(x, draft, w.tau, repeat=2)
    assert gpu["kernel"] == "lm_head_slab_bf16"
    compare(x, draft, w.tau, greedy, gpu)
    check_logits(w, x, tile, x.W)
    # the other epilogues of the same tiles
    dk = tk.planted_drafts(x, 3)
    for k, o in tk.run_topk(x, dk, [1, 3])[0].items():
        tk.check(x, dk, o, k)
    keys = np.random.default_rng(3).integers(0, 2**63, size=(w.B, w.K + 1), dtype=np.uint64)
    ref = oracle.sampled_rows(x.ht, x.W, 1.0, keys.reshape(-1))
    ds = wl.draft_tokens(w, 3, ref[0])

    def scores_row(r):
        return oracle.logits_row(x.ht[r], x.W) + np.array([oracle.gumbel(int(keys.reshape(-1)[r]), v) for v in range(w.V)])
    compare(x, ds, w.tau, ref, run_gpu(x, ds, w.tau, sampled=(1.0, keys)), scores_row=scores_row)


@pytest.mark.parametrize("tile,shape", [
    ((1, 1, 4), dict(B=1, K=9, d_t=1024, d_d=64, V=12300)),         # two lines per slab
    ((2, 6, 4), dict(B=3, K=31, d_t=256, d_d=64, V=20001)),
    ((3, 7, 12), dict(B=4, K=49, d_t=512, d_d=0, V=16389)),          # 200 rows: two row tiles
    ((3, 3, 12), dict(B=1, K=47, d_t=512, d_d=0, V=40001)),
    ((2, 6, 4), dict(B=8, K=32, d_t=512, d_d=64, V=17000)),         # 264 rows: three row tiles
    ((4, 2, 4), dict(B=1, K=20, d_t=1024, d_d=0, V=50177)),         # a last tile that is not full
])
def test_fp8_shapes(tile, shape):
    import paper_2504_20039_amd as aj
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="slab8", p_match=0.6, **shape)
    x = make_inputs(w, 5)
    w8, _ = wl.w_lm_fp8(w, 5)
    x.W = wl.fp8_e4m3_to_bf16_bits(w8)
    greedy = oracle.greedy_rows(x.ht, x.W)
    draft = wl.draft_tokens(w, 5, greedy[0])
    gpu = run_gpu(x, draft, w.tau, repeat=2, w8=w8)
    assert gpu["kernel"] == "lm_head_slab_fp8w"
    compare(x, draft, w.tau, greedy, gpu)
    check_logits(w, x, tile, w8, aj.AJ_W_FP8_E4M3)
