"""Rows whose scores are all -inf.  Finite inputs reach it: products that overflow fp32 downwards, or a large finite inverse
temperature on a row of negative logits.  Every score then attains the maximum, and the token is the lowest one, 0: out_tok
stays in [0, V) through every entry point, both tails and each kind of storage."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def inputs(B, K, d, V, dtype, row_value, seed=4):
    """Rows 1 and K of every window hold row_value in every element, the others N(0, 1); W_lm is negative throughout."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    H = torch.randn(B, K + 1, d, device="cuda", generator=g)
    H[:, 1] = row_value
    H[:, K] = row_value
    W = -(torch.randn(V, d, device="cuda", generator=g).abs() + 0.1) * 1e20
    clf = torch.zeros(d, device="cuda")
    H, W, clf = (t.to(dtype).contiguous() for t in (H, W, clf))
    t = torch.argmax(H.double().view(-1, d) @ W.double().T, dim=1).view(B, K + 1)
    t[:, 1] = t[:, K] = 0
    return H, W, clf, t.to(torch.int32)


SHAPES = [("f32", 2, 7, 64, 300), ("f32", 3, 20, 20, 70), ("f32", 1, 40, 64, 5000), ("bf16", 2, 7, 64, 300), ("bf16", 1, 40, 256, 900),
          ("bf16", 3, 30, 72, 12300)]


@pytest.mark.parametrize("dtype,B,K,d,V", SHAPES)
@pytest.mark.parametrize("call", ["verify", "static", "tree", "topk"])
def test_products_that_overflow(dtype, B, K, d, V, call):
    import torch
    import paper_2504_20039_amd as aj
    H, W, clf, t = inputs(B, K, d, V, torch.float32 if dtype == "f32" else torch.bfloat16, 1e30)
    code = aj.AJ_F32 if dtype == "f32" else aj.AJ_BF16
    flags = aj.AJ_FLAG_TOPK if call == "topk" else 0
    h = aj.aj_create(B, K, d, 0, V, code, 1, flags)
    ol, ot, on = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(3))
    parent = (torch.arange(K, dtype=torch.int32, device="cuda") - 1).expand(B, K).contiguous()
    for draft, want_len in ((t[:, :K].contiguous(), K), (torch.where(torch.arange(K, device="cuda") == 1, 1, t[:, :K]).int().contiguous(), 1)):
        if call == "verify":
            aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.0, ol, ot)
        elif call == "static":
            aj.aj_verify_static(B, K, d, 0, V, code, 1, 0, H, None, W, draft, clf, 0.0, 0.0, ol, ot)
        elif call == "tree":
            aj.aj_verify_tree(h, H, None, W, draft, parent, clf, 0.0, 0.0, ol, ot, on)
        else:
            aj.aj_verify_topk(h, H, W, draft, 1, ol, ot)
        torch.cuda.synchronize()
        assert (ol == want_len).all(), ol
        assert (ot == 0).all(), ot                     # slot 1 and the bonus row are the rows of -inf
        if call != "static":
            t_star, maxlogit, _ = aj.aj_debug_copy(h, B, K, want_score=False)
            assert np.array_equal(t_star.reshape(B, K + 1), t.cpu().numpy())
            assert np.isneginf(maxlogit.reshape(B, K + 1)[:, [1, K]]).all()
    aj.aj_destroy(h)


@pytest.mark.parametrize("dtype,B,K,d,V", SHAPES)
def test_scores_that_the_inverse_temperature_overflows(dtype, B, K, d, V):
    import torch
    import paper_2504_20039_amd as aj
    H, W, clf, t = inputs(B, K, d, V, torch.float32 if dtype == "f32" else torch.bfloat16, 1.0)
    h = aj.aj_create(B, K, d, 0, V, aj.AJ_F32 if dtype == "f32" else aj.AJ_BF16)
    ol, ot = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    keys = torch.arange(B * (K + 1), dtype=torch.int64, device="cuda").view(B, K + 1)
    aj.aj_verify_sampled(h, H, None, W, t[:, :K].contiguous(), clf, 0.0, 1.0, 3e38, keys, ol, ot)
    torch.cuda.synchronize()
    t_star, score, _ = aj.aj_debug_copy(h, B, K, want_score=False)
    aj.aj_destroy(h)
    assert ((t_star >= 0) & (t_star < V)).all()
    rows = [1, K]
    assert (t_star.reshape(B, K + 1)[:, rows] == 0).all() and np.isneginf(score.reshape(B, K + 1)[:, rows]).all()
    assert (ol == K).all() and (ot == 0).all()         # tau = 1 accepts every draft token; the bonus row is one of them
