"""fp32 storage on the bf16 matrix instructions (operands split into three bf16 pieces): every tile that the cost table reaches, at ragged
vocabularies, verify rows and hidden sizes, and values whose pieces the matrix instructions would read as zero."""
import pytest

pytestmark = pytest.mark.gpu

# tile (vocabulary rows, verify rows) <- verify rows, vocabulary, hidden size (1028: ends inside a slab and inside a line)
CASES = [((64, 48), 195, 2768, 1200), ((64, 64), 417, 1961, 1028), ((64, 80), 356, 2877, 1068), ((128, 48), 99, 8501, 1028),
         ((128, 64), 99, 12501, 1028), ((192, 48), 35, 37001, 1028), ((192, 64), 99, 16501, 1028), ((192, 80), 67, 33001, 1028),
         ((128, 80), 67, 16501, 1028), ((256, 48), 35, 49501, 1028), ((256, 64), 99, 25001, 1028), ((256, 80), 131, 25001, 1028),
         ((192, 80), 67, 33024, 2048)]              # whole lines, a last tile that is full


def call(H, W, tile, topk=True):
    import torch
    import paper_2504_20039_amd as aj
    (M, d), V = H.shape, W.shape[0]
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_F32, 1, aj.AJ_FLAG_TOPK, 0)
    assert aj.aj_kernel_name(h) == "lm_head_f32_split"
    assert tile is None or aj.aj_debug_tile(h) == tile
    logits = torch.full((M, V), float("nan"), device="cuda")
    aj.aj_debug_logits(h, H, W, logits)
    torch.cuda.synchronize()
    best = logits.max(1, keepdim=True).values
    t = torch.where(logits == best, torch.arange(V, device="cuda"), V).min(1).values
    draft = t[:M - 1].to(torch.int32).view(1, M - 1).contiguous()
    ol, ot = (torch.full((1,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    aj.aj_verify(h, H, None, W, draft, torch.zeros(d, device="cuda"), 0.0, 0.0, ol, ot)
    t_star, maxlogit, _ = aj.aj_debug_copy(h, 1, M - 1, want_score=False)
    assert (torch.from_numpy(t_star).cuda() == t).all() and (torch.from_numpy(maxlogit).cuda() == best[:, 0]).all()
    assert int(ol) == M - 1 and int(ot) == int(t[M - 1])
    if topk:
        deep = logits[:M - 1].sort(1, descending=True).indices[:, 40:41]
        aj.aj_verify_topk(h, H, W, deep.view(1, M - 1).to(torch.int32).contiguous(), 41 + 5, ol, ot)
        rank = torch.from_numpy(aj.aj_debug_copy_rank(h, 1, M - 1)).cuda()[:M - 1]
    aj.aj_destroy(h)
    return (logits, deep, rank) if topk else logits


@pytest.mark.parametrize("tile,M,V,d", CASES)
def test_tile(tile, M, V, d):
    import torch
    g = torch.Generator(device="cuda").manual_seed(11)
    H, W = torch.randn(M, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g)
    logits, deep, rank = call(H, W, tile)
    exact = H.double() @ W.double().T
    # the bound of the fp32 instructions' test: |sum - exact| <= (d + 1) 2^-24 sum |a b|, sum |a b| <= |a| |b|
    bound = (d + 1) * 2.0**-24 * H.double().norm(dim=1)[:, None] * W.double().norm(dim=1)[None, :]
    assert ((logits.double() - exact).abs() <= bound).all()
    # ... which a lost piece (2^-16 of the products that it takes part in) would still meet: the sums round d / 32 times at random, and
    # the fp32 instructions d / 16 times, 2.9e-7 of the norm at d = 1024
    assert float((logits - exact).norm() / exact.norm()) < 2.9e-7 * (d / 1024) ** 0.5
    slack = 2 * bound[:M - 1].max()
    th = logits[:M - 1].gather(1, deep).double()
    assert (rank >= (logits[:M - 1] > th + slack).sum(1)).all() and (rank <= (logits[:M - 1] >= th - slack).sum(1) - 1).all()


@pytest.mark.parametrize("w,h", [(2.0**-60, 2.0**-60), (2.0**-115, 1.0), (2.0**-126, 1.0), (1.0, 2.0**-120), (2.0**-126, 2.0**100),
                                 (2.0**100, 2.0**-126), (2.0**60, 2.0**60)])
def test_tiny_and_huge_values(w, h):
    import torch
    M, V, d = 67, 16501, 1028
    g = torch.Generator(device="cuda").manual_seed(12)
    H, W = torch.randn(M, d, device="cuda", generator=g) * h, torch.randn(V, d, device="cuda", generator=g) * w
    H[5] = 0                                       # an empty row, and a tile of empty rows, are not tiny ones
    W[256:384] = 0
    H[7] = torch.randn(d, device="cuda", generator=g)
    exact = H.double() @ W.double().T
    logits = call(H, W, (128, 80), topk=False)
    rows = exact.norm(dim=1) > 0
    err = (logits - exact).norm(dim=1)[rows] / exact.norm(dim=1)[rows]
    assert float(err.max()) < 1.5e-6                # d roundings of 2^-24 each at random, and 2.5 times that
    assert (logits[5] == 0).all() and (logits[:, 256:384] == 0).all()


def test_equal_vocabulary_rows_have_equal_logits():
    import torch
    M, V, d = 67, 33001, 2048
    g = torch.Generator(device="cuda").manual_seed(13)
    H, W = torch.randn(M, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g)
    W[-999:] = W[:999]
    logits = call(H, W, None, topk=False)
    assert torch.equal(logits[:, -999:], logits[:, :999])


def split_logits(H, W):
    import torch
    import paper_2504_20039_amd as aj
    (M, d), V = H.shape, W.shape[0]
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_F32)
    name = aj.aj_kernel_name(h)
    logits = torch.full((M, V), float("nan"), device="cuda")
    aj.aj_debug_logits(h, H, W, logits)
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    return name, logits


LONG = 1 + 2.0**-7 - 2.0**-23                       # every bit below the seventh is set


def test_single_products():
    """Logits of one product each: what the six products of pieces leave out is at most 2^-24 of it, and the sum rounds once."""
    import torch
    M, V, d = 67, 16501, 1028
    g = torch.Generator(device="cuda").manual_seed(14)
    H, W = torch.zeros(M, d, device="cuda"), torch.randn(V, d, device="cuda", generator=g)
    x = torch.randn(M, device="cuda", generator=g)
    x[::3] = LONG
    W[::5] = LONG
    W[1::5] = 2 - 2.0**-9 - 2.0**-17 - 2.0**-23
    H[torch.arange(M, device="cuda"), torch.arange(M, device="cuda") * 15] = x
    name, logits = split_logits(H, W)
    assert name == "lm_head_f32_split"
    exact = H.double() @ W.double().T
    assert ((logits - exact).abs() <= (2.0**-23 + 2.0**-29) * exact.abs()).all()


@pytest.mark.parametrize("value", [LONG, 1 + 2.0**-8 - 2.0**-23, 1 + 2.0**-8 + 2.0**-16 - 2.0**-23, 1.5707963, 2 - 2.0**-9 - 2.0**-17 - 2.0**-23])
@pytest.mark.parametrize("d", [256, 1024, 4096])
def test_products_of_one_sign(value, d):
    """What is left out does not add up: where all products are equal the sum is as near as that of the fp32 instructions, to the 2^-24 that
    a product may lack and the sum's last rounding."""
    import torch
    V = 33024
    W = torch.full((V, d), value, device="cuda")
    name, logits = split_logits(torch.full((67, d), value, device="cuda"), W)
    assert name == "lm_head_f32_split"
    name, other = split_logits(torch.full((16, d), value, device="cuda"), W)
    assert name == "lm_head_f32"
    exact = d * float(W[0, 0].double()) ** 2
    err, ref = (float((t.double() / exact - 1).abs().max()) for t in (logits, other))
    assert err <= ref + 2.0**-23


def test_values_that_round_to_infinity():
    """The largest finite values have no bf16 neighbour above: logits that they are part of, and only those, come from the fp32 instructions."""
    import torch
    M, V, d = 67, 16501, 1028
    g = torch.Generator(device="cuda").manual_seed(15)
    big = torch.finfo(torch.float32).max
    H, W = torch.randn(M, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g)
    H[:, 0] = 0
    H[3, 0], H[50, 0], H[7, 1] = 2.0**-40, 2.0**-40, big
    huge = torch.arange(V, device="cuda") % 350 == 0
    plain = split_logits(H, W)[1]
    W[huge, 0] = big
    W[::700, 0] = -big
    name, logits = split_logits(H, W)
    assert name == "lm_head_f32_split"
    exact = H.double() @ W.double().T
    finite = exact.abs() < big
    assert finite[:7].all() and finite[7].any() and not finite[7].all()
    size = H.double().abs() @ W.double().abs().T
    assert ((logits - exact).abs() <= (d + 1) * 2.0**-24 * size)[finite].all()
    assert torch.equal(logits[~finite], torch.copysign(torch.full_like(logits, float("inf")), exact.float())[~finite])
    assert torch.equal(logits[:, ~huge], plain[:, ~huge])


@pytest.mark.parametrize("tile,M,V,d", CASES + [((64, 80), 80, 13001, 4096), ((128, 80), 67, 16501, 4100), ((256, 80), 131, 25001, 2052)])
def test_sums_of_positive_products(tile, M, V, d):
    """Partial sums that grow: each half of the row is summed apart, so that the roundings stay below those of the fp32 instructions."""
    import torch
    import paper_2504_20039_amd as aj
    g = torch.Generator(device="cuda").manual_seed(16)
    H, W = torch.rand(M, d, device="cuda", generator=g), torch.rand(V, d, device="cuda", generator=g)
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_F32)
    got = aj.aj_debug_tile(h)
    aj.aj_destroy(h)
    assert got == tile
    exact = H.double() @ W.double().T
    name, logits = split_logits(H, W)
    assert name == "lm_head_f32_split"
    name, other = split_logits(H[:16].contiguous(), W)
    assert name == "lm_head_f32"
    err, ref = (float((t - exact[:len(t)]).norm() / exact[:len(t)].norm()) for t in (logits, other))
    assert err < ref


def test_rows_of_zeros_take_no_second_pass():
    """Padding of the vocabulary: tiles whose W_lm rows are all zero are not taken for tiles of tiny logits, whose second pass takes longer
    than the whole call."""
    import torch
    import paper_2504_20039_amd as aj
    M, V, d = 68, 32000, 2048
    g = torch.Generator(device="cuda").manual_seed(17)
    H, W = torch.randn(M, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g)
    draft = torch.zeros(1, M - 1, dtype=torch.int32, device="cuda")
    clf = torch.zeros(d, device="cuda")
    ol, ot = (torch.zeros(1, dtype=torch.int32, device="cuda") for _ in range(2))
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_F32)
    assert aj.aj_kernel_name(h) == "lm_head_f32_split"

    def us():
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.5, ol, ot)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        return best

    full = us()
    W[V - 512:] = 0
    W[V - 512::7] = -0.0
    padded = us()
    logits = torch.full((M, V), float("nan"), device="cuda")
    aj.aj_debug_logits(h, H, W, logits)
    # one value in such a tile that the matrix instructions read as zero, and its logits are exact again
    W[V - 100, 5] = 2.0**-140
    aj.aj_debug_logits(h, H, W, tiny := torch.full((M, V), float("nan"), device="cuda"))
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    assert (logits[:, V - 512:] == 0).all()
    assert padded < 1.5 * full                      # 3.4 times with the second pass
    assert torch.equal(tiny[:, V - 100], H[:, 5] * 2.0**-140)
