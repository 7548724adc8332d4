"""fp32 storage at the edges of its tiles: every number of 16-row blocks, vocabularies that select 1 to 4 vocabulary blocks per
tile (all pairs: test_gpu_tiles.py), hidden sizes that end inside a 32-element step, through every entry point's epilogue."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import compare, make_inputs, parity_case, run_gpu
import test_gpu_topk as tk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,shape", [              # tile: vocabulary blocks and verify-row blocks of 16
    ((1, 1), dict(B=1, K=1, d_t=4, d_d=0, V=5)),                 # the smallest call: three of the four waves have no step
    ((1, 1), dict(B=1, K=8, d_t=20, d_d=4, V=17)),               # one ragged step; a second vocabulary tile of one row
    ((2, 1), dict(B=2, K=7, d_t=132, d_d=64, V=4100)),
    ((2, 2), dict(B=1, K=16, d_t=1000, d_d=128, V=4097)),        # 17 rows; a last tile of one vocabulary row
    ((3, 3), dict(B=3, K=15, d_t=516, d_d=64, V=8200)),
    ((3, 4), dict(B=4, K=15, d_t=256, d_d=64, V=16500)),
    ((3, 5), dict(B=4, K=19, d_t=260, d_d=0, V=17000)),
    ((2, 3), dict(B=3, K=26, d_t=128, d_d=64, V=2050)),          # 81 rows: two row tiles
    ((3, 3), dict(B=9, K=31, d_t=96, d_d=64, V=9001)),           # 288 rows: six row tiles
    ((4, 1), dict(B=1, K=9, d_t=68, d_d=0, V=12545)),            # a last tile of one vocabulary row
    ((4, 5), dict(B=3, K=25, d_t=100, d_d=4, V=16001)),          # the largest tile, ragged on every side
])
def test_f32_shapes(tile, shape):
    import torch
    import paper_2504_20039_amd as aj
    w = wl.scaled(wl.WORKLOADS["tiny_f32"], name="f32", p_match=0.6, **shape)
    rep, x, draft, greedy, gpu = parity_case(w, 3, repeat=2)
    h = aj.aj_create(w.B, w.K, w.d_t, w.d_d, w.V, aj.AJ_F32)
    assert aj.aj_debug_tile(h) == (16 * tile[0], 16 * tile[1])
    logits = torch.empty((w.M, w.V), dtype=torch.float32, device="cuda")
    aj.aj_debug_logits(h, aj.device_tensor(x.ht), aj.device_tensor(x.W), logits)
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    # |fp32 sum of d products - exact| <= d 2^-24 sum |a b| (any order); sum |a b| <= |a| |b|
    bound = (w.d_t + 1) * 2.0**-24 * np.linalg.norm(x.ht, axis=1)[:, None] * np.linalg.norm(x.W, axis=1)[None, :]
    assert (np.abs(logits.cpu().numpy() - x.ht.astype(np.float64) @ x.W.astype(np.float64).T) <= bound).all()
    # the other epilogues of the same tiles
    dk = tk.planted_drafts(x, 3)
    for k, o in tk.run_topk(x, dk, [1, 3])[0].items():
        tk.check(x, dk, o, k)
    keys = np.random.default_rng(3).integers(0, 2**63, size=(w.B, w.K + 1), dtype=np.uint64)
    ref = oracle.sampled_rows(x.ht, x.W, 1.0, keys.reshape(-1))
    ds = wl.draft_tokens(w, 3, ref[0])
    gpu = run_gpu(x, ds, w.tau, sampled=(1.0, keys))

    def scores_row(r):
        return oracle.logits_row(x.ht[r], x.W) + np.array([oracle.gumbel(int(keys.reshape(-1)[r]), v) for v in range(w.V)])
    compare(x, ds, w.tau, ref, gpu, scores_row=scores_row)


@pytest.mark.parametrize("tile,shape", [
    ((3, 2), dict(B=1, K=16, d_t=260, d_d=0, V=16417)),          # 17 rows; a last tile of one vocabulary row
    ((3, 3), dict(B=3, K=26, d_t=96, d_d=64, V=8208)),           # two row tiles, the vocabulary exactly full
    ((3, 5), dict(B=2, K=39, d_t=64, d_d=4, V=16450)),
])
def test_f32_three_block_tiles(tile, shape):
    test_f32_shapes(tile, shape)


@pytest.mark.parametrize("B,K,d,V", [
    (4, 19, 14_000_004, 5),            # 80 verify rows: row 77 begins beyond 2^32 bytes
    (1, 1, 17_500_000, 70),            # 70 vocabulary rows: row 62 does
])
def test_f32_rows_whose_offsets_pass_32_bits(B, K, d, V):
    """Every verify row is one unit vector, so its logits are the W_lm column it picks, exactly."""
    import torch
    import paper_2504_20039_amd as aj
    M = B * (K + 1)
    g = torch.Generator(device="cuda").manual_seed(5)
    W = torch.randn(V, d, device="cuda", generator=g)
    H = torch.zeros(M, d, device="cuda")
    pick = torch.randint(0, d, (M,), device="cuda", generator=g)
    pick[0], pick[M - 1] = 0, d - 1
    H[torch.arange(M, device="cuda"), pick] = 1.0
    want = W[:, pick].T.contiguous()
    t = want.argmax(1).to(torch.int32).view(B, K + 1)
    draft = t[:, :K].contiguous()
    clf = torch.zeros(d, device="cuda")
    ol, ot = (torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    logits = torch.full((M, V), float("nan"), device="cuda")
    h = aj.aj_create(B, K, d, 0, V, aj.AJ_F32)
    aj.aj_debug_logits(h, H, W, logits)
    aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.5, ol, ot)
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    assert torch.equal(logits, want)
    assert (ol == K).all() and torch.equal(ot, t[:, K])


@pytest.mark.parametrize("B,K,V", [(64, 999, 720), (1000, 177, 153)])
def test_f32_static_entry_takes_what_tiles_of_64_rows_fit(B, K, V):
    """Many rows of a small vocabulary: 64-row tiles need 6.9 and 6.4 MB of partials, the 48- and 32-row tiles that fill the
    compute units better would need more than the static array's 8 MiB."""
    import torch
    import paper_2504_20039_amd as aj
    d, M = 16, B * (K + 1)
    g = torch.Generator(device="cuda").manual_seed(6)
    H = torch.randn(M, d, device="cuda", generator=g)
    W = torch.randn(V, d, device="cuda", generator=g)
    draft = torch.randint(0, V, (B, K), device="cuda", generator=g, dtype=torch.int32)
    clf = torch.zeros(d, device="cuda")
    out = [torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(4)]
    h = aj.aj_create(B, K, d, 0, V, aj.AJ_F32)
    aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.0, out[2], out[3])
    t_star = aj.aj_debug_copy(h, B, K, want_score=False)[0].reshape(B, K + 1)
    draft[:, :3] = torch.from_numpy(t_star[:, :3]).cuda()
    aj.aj_verify(h, H, None, W, draft, clf, 0.0, 0.0, out[2], out[3])
    aj.aj_verify_static(B, K, d, 0, V, aj.AJ_F32, 1, 0, H, None, W, draft, clf, 0.0, 0.0, out[0], out[1])
    torch.cuda.synchronize()
    aj.aj_destroy(h)
    assert (out[0] >= 3).all() and torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])


def test_f32_vocabularies_beyond_the_limit_are_refused():
    import paper_2504_20039_amd as aj
    for B in (0, 1):
        aj.aj_destroy(aj.aj_create(B, 1, 4, 0, 65535 * 64, aj.AJ_F32))
        with pytest.raises(aj.AjError) as e:
            aj.aj_create(B, 1, 4, 0, 65535 * 64 + 1, aj.AJ_F32)
        assert e.value.status == -1


@pytest.mark.parametrize("V", [5, 100, 128])               # 1, 7 and 8 vocabulary tiles of 16 rows, six row tiles
def test_f32_few_vocabulary_tiles(V):
    test_f32_shapes((1, 3), dict(B=9, K=31, d_t=68, d_d=4, V=V))
