"""Equal W_lm rows (padding, untrained tokens) have equal logits wherever they lie in the vocabulary, so the lowest of them is the
greedy token.  The small-tile kernel keeps that rule where it replaced a kernel that sums all rows in one order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,d,V,fp8", [
    (3, 20, 2888, 20001, False),       # a hidden size no other kernel takes
    (1, 16, 1000, 50257, False),
    (10, 49, 1000, 13000, False),      # 500 rows: several row tiles
    (3, 20, 1120, 24000, False),       # a multiple of 32
    (4, 19, 1600, 24000, False),       # a multiple of 64
    (3, 49, 1088, 16000, False),       # 150 rows
    (6, 32, 1024, 16000, False),       # 198 rows
    (8, 32, 2048, 17000, False),       # 264 rows
    (6, 32, 2048, 17000, True),
])
def test_the_lowest_of_equal_rows_wins(B, K, d, V, fp8):
    import torch
    import paper_2504_20039_amd as aj
    M, n = B * (K + 1), 64
    g = torch.Generator(device="cuda").manual_seed(7)
    W = torch.randn(V, d, device="cuda", generator=g).to(torch.float8_e4m3fn if fp8 else torch.bfloat16)
    perm = torch.randperm(V, device="cuda", generator=g)[:3 * n].view(3, n).sort(0).values     # n rows, three equal copies of each
    W = W.view(torch.uint8) if fp8 else W
    W[perm[1]] = W[perm[0]]
    W[perm[2]] = W[perm[0]]
    owner = torch.arange(M, device="cuda") % n
    wide = (W.view(torch.float8_e4m3fn) if fp8 else W)[perm[0]].float()
    H = (torch.randn(M, d, device="cuda", generator=g) + wide[owner] * 0.5).to(torch.bfloat16)
    want = perm[0][owner].to(torch.int32)
    h = aj.aj_create(B, K, d, 0, V, aj.AJ_BF16, 1, 0, 0, aj.AJ_W_FP8_E4M3 if fp8 else aj.AJ_W_SAME)
    assert "slab" in aj.aj_kernel_name(h)
    logits = torch.empty(M, V, device="cuda")
    aj.aj_debug_logits(h, H, W, logits)
    ol, ot = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    clf = torch.zeros(d, device="cuda", dtype=torch.bfloat16)
    draft = want.view(B, K + 1)[:, :K].contiguous()
    aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.0, ol, ot)
    torch.cuda.synchronize()
    t_star = aj.aj_debug_copy(h, B, K, want_score=False)[0]
    aj.aj_destroy(h)
    assert torch.equal(logits[:, perm[0]], logits[:, perm[1]]) and torch.equal(logits[:, perm[0]], logits[:, perm[2]])
    assert np.array_equal(t_star, want.cpu().numpy())
    assert (ol == K).all() and torch.equal(ot, want.view(B, K + 1)[:, K])
