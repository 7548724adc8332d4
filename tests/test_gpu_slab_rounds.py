"""Small tiles in more than one round: 4 waves of several blocks, tiles of uneven heights (the waves' rows end inside a block of 16),
one and several row tiles; last tiles that are full and that hold one vocabulary row.  (One round, waves of one block: the shapes of
test_gpu_tiles.py.)"""
import pytest

from parity import check_small_tile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,nb,mb,M,V,d", [
    ("bf16", 2, 2, 19, 147501, 328),
    ("bf16", 2, 3, 35, 147501, 328),
    ("bf16", 2, 6, 259, 20713, 328),         # three row tiles
    ("bf16", 2, 7, 387, 12301, 328),
    ("bf16", 2, 8, 227, 24919, 328),
    ("bf16", 3, 2, 19, 82401, 328),
    ("bf16", 3, 3, 35, 82001, 328),
    ("bf16", 3, 4, 51, 82001, 328),
    ("bf16", 3, 5, 131, 33331, 328),
    ("bf16", 3, 6, 163, 33331, 328),
    ("bf16", 3, 7, 291, 22001, 328),
    ("bf16", 3, 8, 115, 65577, 328),
    ("bf16", 4, 1, 3, 114801, 328),
    ("bf16", 4, 2, 19, 98524, 328),
    ("bf16", 4, 3, 35, 98524, 328),
    ("bf16", 4, 4, 51, 98524, 328),
    ("bf16", 4, 5, 131, 49201, 328),
    ("bf16", 4, 6, 83, 98524, 328),
    ("bf16", 1, 1, 11, 20011, 328),          # two rounds of the smallest tile
    ("fp8", 2, 3, 35, 147601, 4096),
    ("fp8", 2, 4, 51, 49201, 4096),
    ("fp8", 2, 5, 131, 24919, 512),
    ("fp8", 2, 6, 259, 15401, 512),
    ("fp8", 2, 7, 195, 24919, 512),
    ("fp8", 2, 8, 227, 24919, 512),
    ("fp8", 3, 3, 35, 131201, 4096),
    ("fp8", 3, 4, 51, 131201, 4096),
    ("fp8", 3, 5, 147, 65601, 512),
    ("fp8", 3, 6, 259, 21601, 512),
    ("fp8", 3, 7, 195, 65601, 512),
    ("fp8", 3, 8, 115, 72011, 512),
])
def test_rounds(storage, nb, mb, M, V, d):
    import torch
    import paper_2504_20039_amd as aj
    g = torch.Generator(device="cuda").manual_seed(17)
    H = torch.randn(M, d, device="cuda", generator=g).bfloat16()
    W = torch.randn(V, d, device="cuda", generator=g).to(torch.float8_e4m3fn if storage == "fp8" else torch.bfloat16)
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_BF16, 1, 0, 0, aj.AJ_W_FP8_E4M3 if storage == "fp8" else aj.AJ_W_SAME)
    assert aj.aj_kernel_name(h) == {"bf16": "lm_head_slab_bf16", "fp8": "lm_head_slab_fp8w"}[storage]
    check_small_tile(h, nb, mb, 4)
    check_call(h, storage, H, W)


def check_call(h, storage, H, W):
    """Logits, greedy tokens and outputs of a handle, which it destroys."""
    import torch
    import paper_2504_20039_amd as aj
    (M, d), V = H.shape, W.shape[0]
    data = W.view(torch.uint8) if storage == "fp8" else W
    logits = torch.full((M, V), float("nan"), device="cuda")
    aj.aj_debug_logits(h, H, data, logits)
    torch.cuda.synchronize()
    exact = H.double() @ W.float().double().T
    # |fp32 sum of d products - exact| <= d 2^-24 sum |a b| in any order; sum |a b| <= |a| |b|
    bound = (d + 1) * 2.0**-24 * H.double().norm(dim=1)[:, None] * W.float().double().norm(dim=1)[None, :]
    assert ((logits.double() - exact).abs() <= bound).all()
    best = logits.max(1, keepdim=True).values
    t = torch.where(logits == best, torch.arange(V, device="cuda"), V).min(1).values
    draft = t[:M - 1].to(torch.int32).view(1, M - 1).contiguous()
    ol, ot = (torch.full((1,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    aj.aj_verify(h, H, None, data, draft, torch.zeros(d, device="cuda", dtype=torch.bfloat16), 0.0, 0.0, ol, ot)
    t_star, maxlogit, _ = aj.aj_debug_copy(h, 1, M - 1, want_score=False)
    aj.aj_destroy(h)
    assert (torch.from_numpy(t_star).cuda() == t).all() and (torch.from_numpy(maxlogit).cuda() == best[:, 0]).all()
    assert int(ol) == M - 1 and int(ot) == int(t[M - 1])


@pytest.mark.parametrize("storage,M,V,height", [
    ("bf16", 63, 12324, 52), ("bf16", 200, 12376, 104), ("bf16", 63, 32868, 132), ("bf16", 63, 49296, 208), ("bf16", 261, 15400, 200),
    ("bf16", 261, 20584, 124), ("bf16", 261, 21516, 132), ("fp8", 93, 12324, 52), ("fp8", 261, 21516, 132),
])
@pytest.mark.parametrize("last", ["full", "one row"])
def test_last_tile(storage, M, V, height, last):
    import torch
    import paper_2504_20039_amd as aj
    V, d = V + (last == "one row"), 512 if storage == "fp8" else 328
    g = torch.Generator(device="cuda").manual_seed(18)
    H = torch.randn(M, d, device="cuda", generator=g).bfloat16()
    W = torch.randn(V, d, device="cuda", generator=g).to(torch.float8_e4m3fn if storage == "fp8" else torch.bfloat16)
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_BF16, 1, 0, 0, aj.AJ_W_FP8_E4M3 if storage == "fp8" else aj.AJ_W_SAME)
    assert "slab" in aj.aj_kernel_name(h)
    assert aj.aj_debug_tile(h)[0] == height and V % height == (last == "one row")
    check_call(h, storage, H, W)
