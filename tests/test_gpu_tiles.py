"""Every tile that the fp32 and the small-tile kernel choose by shape, each at a ragged vocabulary and a ragged number of verify
rows: all logits against the fp64 product, the greedy tokens and the top-K ranks against those logits.  The tile, its waves and its k order
are asserted, so that a change of the cost tables cannot leave one untested unseen.  (Tiles of four vocabulary blocks and more than three row blocks are never
the cheapest with FP8 weights, nor are two or three vocabulary blocks with one row block in bf16.)"""
import pytest

from parity import check_small_tile

pytestmark = pytest.mark.gpu

VOCAB = {"f32": {1: 1001, 2: 4508, 3: 8516, 4: 12524}, "bf16": {1: 12289, 2: 16798, 3: 33040, 4: 50091},
         "fp8": {1: 12289, 2: 16798, 3: 33040, 4: 50091}}
CASES = [("f32", nb, mb) for nb in (1, 2, 3, 4) for mb in (1, 2, 3, 4, 5)] + \
        [("bf16", nb, mb) for nb, mbs in ((1, range(1, 5)), (2, range(2, 9)), (3, range(2, 9)), (4, range(1, 7))) for mb in mbs] + \
        [("fp8", nb, mb) for nb, mbs in ((1, range(1, 5)), (2, range(1, 9)), (3, range(1, 9)), (4, range(1, 4))) for mb in mbs]


@pytest.mark.parametrize("storage,nb,mb", CASES)
def test_tile(storage, nb, mb):
    import torch
    import paper_2504_20039_amd as aj
    M, V = 16 * mb - 13, VOCAB[storage][nb]
    d = {"f32": 68, "bf16": 328, "fp8": 1024}[storage]
    if nb == 2 and mb > 4 and storage != "f32":
        V = 12289
    if (storage, nb, mb) == ("fp8", 3, 8):
        M, V = 225, 16798                                 # two row tiles of eight blocks
    g = torch.Generator(device="cuda").manual_seed(11)
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    H = torch.randn(M, d, device="cuda", generator=g).to(dt)
    W = torch.randn(V, d, device="cuda", generator=g).to(torch.float8_e4m3fn if storage == "fp8" else dt)
    wide = W.double() if storage != "fp8" else W.float().double()
    W = W.view(torch.uint8) if storage == "fp8" else W
    topk = storage != "fp8"
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_F32 if storage == "f32" else aj.AJ_BF16, 1, aj.AJ_FLAG_TOPK if topk else 0, 0,
                     aj.AJ_W_FP8_E4M3 if storage == "fp8" else aj.AJ_W_SAME)
    assert aj.aj_kernel_name(h) == {"f32": "lm_head_f32", "bf16": "lm_head_slab_bf16", "fp8": "lm_head_slab_fp8w"}[storage]
    if storage == "f32":
        assert aj.aj_debug_tile(h) == (16 * nb, 16 * mb)
    elif storage == "bf16":
        check_small_tile(h, nb, mb, {1: 4, 2: 8, 3: 12, 4: 16 if mb <= 4 else 8}[nb], order=0)
    else:
        check_small_tile(h, nb, mb, {1: 4, 2: 8, 3: 12}[nb] if mb > 2 and nb < 4 and (nb, mb) != (2, 6) else 4, order=2 if M <= 112 else 0)

    logits = torch.full((M, V), float("nan"), device="cuda")
    aj.aj_debug_logits(h, H, W, logits)
    torch.cuda.synchronize()
    exact = H.double() @ wide.T
    # |fp32 sum of d products - exact| <= d 2^-24 sum |a b| in any order (fp32 products: one more rounding each); sum |a b| <= |a| |b|
    bound = (d + 1) * 2.0**-24 * H.double().norm(dim=1)[:, None] * wide.norm(dim=1)[None, :]
    assert ((logits.double() - exact).abs() <= bound).all()

    index = torch.arange(V, device="cuda")
    best = logits.max(1, keepdim=True).values
    t = torch.where(logits == best, index, V).min(1).values
    draft = t[:M - 1].to(torch.int32).view(1, M - 1).contiguous()
    ol, ot = (torch.full((1,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    aj.aj_verify(h, H, None, W, draft, torch.zeros(d, device="cuda", dtype=dt), 0.0, 0.0, ol, ot)
    t_star, maxlogit, _ = aj.aj_debug_copy(h, 1, M - 1, want_score=False)
    assert (torch.from_numpy(t_star).cuda() == t).all() and (torch.from_numpy(maxlogit).cuda() == best[:, 0]).all()
    assert int(ol) == M - 1 and int(ot) == int(t[M - 1])
    if topk:
        deep = logits[:M - 1].sort(1, descending=True).indices[:, 40:41]
        aj.aj_verify_topk(h, H, W, deep.view(1, M - 1).to(torch.int32).contiguous(), 41 + 5, ol, ot)
        rank = torch.from_numpy(aj.aj_debug_copy_rank(h, 1, M - 1)).cuda()[:M - 1]
        # the token's own logit is a separate dot product: entries within the two sums' rounding may fall on either side
        slack = 2 * bound[:M - 1].max()
        th = logits[:M - 1].gather(1, deep).double()
        assert (rank >= (logits[:M - 1] > th + slack).sum(1)).all() and (rank <= (logits[:M - 1] >= th - slack).sum(1) - 1).all()
    aj.aj_destroy(h)
