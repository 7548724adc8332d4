"""Every entry point on the fp32 kernel that runs on the bf16 matrix instructions: greedy, top-K, sampled, tree and static calls against the
oracle, its second pass under a sampling key, and rows whose scores are all -inf."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import compare, make_inputs, run_gpu
from test_gpu_f32 import test_f32_shapes as check_shape
from test_gpu_overflow import test_products_that_overflow as check_products
from test_gpu_overflow import test_scores_that_the_inverse_temperature_overflows as check_scores
import test_gpu_tree as tree

pytestmark = pytest.mark.gpu

SHAPE = dict(B=3, K=22, d_t=260, d_d=64, V=33001)            # 69 rows: tiles of 192 x 80, the last of 169 vocabulary rows


def workload(**more):
    return wl.scaled(wl.WORKLOADS["tiny_f32"], name="split", p_match=0.6, **{**SHAPE, **more})


def kernel_of(B, K, d, V):
    import paper_2504_20039_amd as aj
    h = aj.aj_create(B, K, d, 0, V, aj.AJ_F32)
    name = aj.aj_kernel_name(h)
    aj.aj_destroy(h)
    return name


def test_greedy_topk_and_sampled():
    assert kernel_of(3, 22, 260, 33001) == "lm_head_f32_split"
    check_shape((12, 5), SHAPE)


@pytest.mark.parametrize("shape", ["chain", "bushy"])
def test_tree(shape):
    w = workload()
    x = make_inputs(w, 4)
    greedy = oracle.greedy_rows(x.ht, x.W)
    rng = np.random.default_rng(4)
    parent = tree.random_trees(rng, w.B, w.K, shape)
    draft = tree.tree_drafts(rng, greedy[0].reshape(w.B, w.K + 1), parent, w.V, 0.7)
    tree.check(x, draft, parent, 0.5, tree.run_tree(x, draft, parent, 0.5), greedy)


def test_static():
    import torch
    import paper_2504_20039_amd as aj
    w = workload()
    x = make_inputs(w, 5)
    draft = wl.draft_tokens(w, 5, oracle.greedy_rows(x.ht, x.W)[0])
    gpu = run_gpu(x, draft, w.tau)
    assert gpu["kernel"] == "lm_head_f32_split"
    dev = [aj.device_tensor(a) for a in (x.ht, x.hd, x.W, np.ascontiguousarray(draft, np.int32), x.cw)]
    ol, ot = (torch.full((w.B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    aj.aj_verify_static(w.B, w.K, w.d_t, w.d_d, w.V, aj.AJ_F32, 1, 0, *dev, w.clf_b, w.tau, ol, ot)
    torch.cuda.synchronize()
    assert np.array_equal(ol.cpu().numpy(), gpu["out_len"]) and np.array_equal(ot.cpu().numpy(), gpu["out_tok"])


def test_sampled_second_pass():
    """Rows of tiny hidden states, whose tiles are computed again, under a temperature at which their logits count next to the noise."""
    w = workload()
    x = make_inputs(w, 6)
    x.ht = np.array(x.ht, np.float32).reshape(w.M, w.d_t)
    x.ht[::4] *= np.float32(2.0**-110)
    inv_temp = 2.0**114        # logits of standard deviation 0.02 sqrt(260) 2^4 = 5: at 2^110 the noise decides every row, far above none
    keys = np.random.default_rng(6).integers(0, 2**63, size=(w.B, w.K + 1), dtype=np.uint64)
    ref = oracle.sampled_rows(x.ht, x.W, inv_temp, keys.reshape(-1))
    draft = wl.draft_tokens(w, 6, ref[0])
    gpu = run_gpu(x, draft, w.tau, sampled=(inv_temp, keys))
    assert gpu["kernel"] == "lm_head_f32_split"

    def scores_row(r):
        noise = np.array([oracle.gumbel(int(keys.reshape(-1)[r]), v) for v in range(w.V)])
        return oracle.logits_row(x.ht[r], x.W) * inv_temp + noise
    compare(x, draft, w.tau, ref, gpu, scores_row=scores_row)
    # the noise decided some of those rows, and the logits others
    plain = oracle.greedy_rows(x.ht, x.W)[0]
    assert 0 < (plain[::4] != ref[0][::4]).sum() < len(plain[::4])


@pytest.mark.parametrize("call", ["verify", "static", "tree", "topk"])
def test_rows_of_minus_infinity(call):
    assert kernel_of(2, 33, 256, 33024) == "lm_head_f32_split"
    check_products("f32", 2, 33, 256, 33024, call)


def test_scores_of_minus_infinity():
    check_scores("f32", 2, 33, 256, 33024)
