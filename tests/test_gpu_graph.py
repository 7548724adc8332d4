"""aj_verify and aj_verify_static enqueue kernels only (no allocation, no memset, no synchronisation), so a caller can
capture them in a HIP graph.  A graph of one call is replayed several times, with the program's own eager work and
synchronisations between the replays and with new inputs written into the captured buffers, and every replay is checked
against the eager call on the same inputs."""
import numpy as np
import pytest

import workloads as wl
from parity import make_inputs, oracle_greedy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,static", [
    (dict(B=1, K=16, d_t=4096, d_d=64, V=5003), False),      # one-launch tail, 16-row-tile kernel
    (dict(B=1, K=64, d_t=1024, d_d=64, V=9000), False),      # split tail, accumulator-resident kernel
    (dict(B=4, K=32, d_t=512, d_d=64, V=3000), False),       # wide kernel
    (dict(B=4, K=32, d_t=512, d_d=64, V=3000), True),        # the entry point that allocates nothing
])
def test_a_captured_call_replays_like_the_eager_one(shape, static):
    import torch
    import paper_2504_20039_amd as aj
    w = wl.scaled(wl.WORKLOADS["8b_b1_k16"], name="graph", p_match=0.85, **shape)
    x = make_inputs(w, 11)
    greedy = oracle_greedy(x)
    drafts = [np.ascontiguousarray(wl.draft_tokens(w, seed, greedy[0]), np.int32) for seed in (11, 12, 13)]
    ht, hd, W, cw = (aj.device_tensor(a) for a in (x.ht, x.hd, x.W, x.cw))
    d_draft = aj.device_tensor(drafts[0])
    h = None if static else aj.aj_create(w.B, w.K, w.d_t, w.d_d, w.V, w.dtype_code, 1, 0, 0)

    def call(draft, ol, ot):
        if static:
            aj.aj_verify_static(w.B, w.K, w.d_t, w.d_d, w.V, w.dtype_code, 1, 0, ht, hd, W, draft, cw, w.clf_b, w.tau, ol, ot)
        else:
            aj.aj_verify(h, ht, hd, W, draft, cw, w.clf_b, w.tau, ol, ot)

    try:
        eager = []
        for dr in drafts:
            ol = torch.full((w.B,), -7, dtype=torch.int32, device="cuda")
            ot = torch.full((w.B,), -7, dtype=torch.int32, device="cuda")
            call(aj.device_tensor(dr), ol, ot)
            torch.cuda.synchronize()
            eager.append((ol.cpu().numpy().copy(), ot.cpu().numpy().copy()))
        if w.B >= 4:      # (the replays below are told apart by their results)
            assert any(not np.array_equal(eager[0][0], e[0]) or not np.array_equal(eager[0][1], e[1]) for e in eager[1:])

        g_len = torch.full((w.B,), -7, dtype=torch.int32, device="cuda")
        g_tok = torch.full((w.B,), -7, dtype=torch.int32, device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            call(d_draft, g_len, g_tok)              # a warm-up on the capture stream
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(d_draft, g_len, g_tok)
        for rnd in range(2):
            for i, dr in enumerate(drafts):
                d_draft.copy_(torch.from_numpy(dr).cuda())
                g_len.fill_(-7)                      # eager work of the program between the replays
                g_tok.fill_(-7)
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert np.array_equal(g_len.cpu().numpy(), eager[i][0]), (rnd, i)
                assert np.array_equal(g_tok.cpu().numpy(), eager[i][1]), (rnd, i)
    finally:
        if h is not None:
            aj.aj_destroy(h)


@pytest.mark.parametrize("dtype,tree,B,K,d_t,V,kernel", [
    ("bf16", False, 2, 40, 1000, 12300, "lm_head_slab_bf16"),      # small tiles, split tail
    ("bf16", True, 2, 40, 1000, 12300, "lm_head_slab_bf16"),       # ... and the two kernels of a draft tree's split form
    ("bf16", True, 3, 100, 512, 3000, None),                       # nodes of more than one wave
    ("f32", False, 4, 16, 260, 4100, "lm_head_f32"),
    ("f32", True, 2, 12, 260, 4100, "lm_head_f32"),                # one-launch tree tail
])
def test_captured_trees_and_small_tiles_replay_like_the_eager_call(dtype, tree, B, K, d_t, V, kernel):
    import torch
    import paper_2504_20039_amd as aj
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(3)
    H = torch.randn(B * (K + 1), d_t, device="cuda", generator=g).to(dt)
    W = (torch.randn(V, d_t, device="cuda", generator=g) * 0.02).to(dt)
    clf = (torch.randn(d_t, device="cuda", generator=g) * d_t ** -0.5).to(dt)
    span = torch.arange(K, device="cuda")
    parent = ((torch.rand(B, K, device="cuda", generator=g) * (span + 1)).long().clamp(max=span) - 1).to(torch.int32).contiguous()
    h = aj.aj_create(B, K, d_t, 0, V, aj.AJ_F32 if dtype == "f32" else aj.AJ_BF16)
    if kernel:
        assert aj.aj_kernel_name(h) == kernel
    out = [torch.full((B,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
    d_draft = torch.zeros(B, K, dtype=torch.int32, device="cuda")

    def call():
        if tree:
            aj.aj_verify_tree(h, H, None, W, d_draft, parent, clf, 0.0, 0.5, *out)
        else:
            aj.aj_verify(h, H, None, W, d_draft, clf, 0.0, 0.5, out[0], out[1])

    call()
    t = torch.from_numpy(aj.aj_debug_copy(h, B, K, want_score=False)[0]).cuda().view(B, K + 1)
    right = t.gather(1, parent.long() + 1) if tree else t[:, :K]
    drafts, eager = [], []
    for share in (0.3, 0.9, 0.98):
        wrong = torch.rand(B, K, device="cuda", generator=g) > share
        drafts.append(torch.where(wrong, (right + 1) % V, right).to(torch.int32))
        d_draft.copy_(drafts[-1])
        call()
        torch.cuda.synchronize()
        eager.append([o.clone() for o in out])
    assert not all(torch.equal(eager[0][0], e[0]) for e in eager[1:])      # the replays are told apart by their results
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(2):
        for dr, want in zip(drafts, eager):
            d_draft.copy_(dr)
            for o in out:
                o.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for o, e in zip(out[:3 if tree else 2], want):
                assert torch.equal(o, e)
    aj.aj_destroy(h)
