"""Large tiles of 160, 192 and 224 verify rows: one and several blocks of k, row and vocabulary tiles that end after one row, through every
entry point's epilogue; and the rows at which two row tiles replace the wide kernel."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import compare, make_inputs, run_gpu
from test_gpu_parity import oracle_greedy
from test_gpu_slab import logit_bound
import test_gpu_topk as tk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_blocks,shape", [
    (5, dict(B=3, K=106, d_t=256, d_d=64, V=12289)),       # 321 rows: the third row tile holds one; a last vocabulary tile of one row
    (5, dict(B=2, K=159, d_t=1024, d_d=0, V=12544)),       # 320 rows and 49 vocabulary tiles, exactly
    (6, dict(B=9, K=88, d_t=512, d_d=64, V=12289)),        # 801 rows
    (7, dict(B=31, K=30, d_t=256, d_d=64, V=12289)),       # 961 rows
    (7, dict(B=7, K=142, d_t=768, d_d=0, V=12400)),
    (5, dict(B=8, K=24, d_t=1024, d_d=64, V=32768)),       # 200 rows: two row tiles, 256 tiles in all
])
def test_row_tiles(row_blocks, shape):
    import torch
    import paper_2504_20039_amd as aj
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="rows", p_match=0.6, **shape)
    x = make_inputs(w, 3)
    greedy = oracle_greedy(x)
    draft = wl.draft_tokens(w, 3, greedy[0])
    gpu = run_gpu(x, draft, w.tau, repeat=2)
    assert gpu["kernel"] == f"lm_head_pair{row_blocks}_bf16"
    compare(x, draft, w.tau, greedy, gpu)
    h = aj.aj_create(w.B, w.K, w.d_t, w.d_d, w.V, aj.AJ_BF16)
    logits = torch.empty((w.M, w.V), dtype=torch.float32, device="cuda")
    aj.aj_debug_logits(h, aj.device_tensor(x.ht), aj.device_tensor(x.W), logits)
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    ref = wl.widen(x.ht).astype(np.float64) @ wl.widen(x.W).astype(np.float64).T
    assert (np.abs(logits.cpu().numpy() - ref) <= logit_bound(w, x)).all()
    dk = tk.planted_drafts(x, 3)
    for k, o in tk.run_topk(x, dk, [1, 3])[0].items():
        tk.check(x, dk, o, k)
    keys = np.random.default_rng(3).integers(0, 2**63, size=(w.B, w.K + 1), dtype=np.uint64)
    ref = oracle.sampled_rows(x.ht, x.W, 1.0, keys.reshape(-1))
    ds = wl.draft_tokens(w, 3, ref[0])

    def scores_row(r):
        return oracle.logits_row(x.ht[r], x.W) + np.array([oracle.gumbel(int(keys.reshape(-1)[r]), v) for v in range(w.V)])
    compare(x, ds, w.tau, ref, run_gpu(x, ds, w.tau, sampled=(1.0, keys)), scores_row=scores_row)
