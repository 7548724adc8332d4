"""Performance cases of the verification step: the calls that a speculative-decoding server makes, through the public
entry points of the library, over the range of sizes, storage types and options they are made with.

A case is one configuration of one entry point (``op``) with the sizes of its speculation windows; ``prepare`` makes
what the server holds before the call (hidden states, LM head, judge, draft tokens, a handle), ``run`` is the call.

Inputs follow the recipe of the synthetic workloads (unit-RMS hidden states, LM-head entries N(0, 0.02^2), judge
weights N(0, 1/D), draft tokens that match with probability ``p_match``), with one addition: as in a trained model every
verify row has a clear favourite token and a clear second one, several standard deviations above the rest.  They are
planted by adding a small multiple of the row's hidden state to two LM-head rows, so the draft tokens can be drawn
without running the path first, and a mismatching draft token is the second choice half of the time.
"""
from __future__ import annotations

import math

import torch

import paper_2504_20039_amd as aj

DEVICE = "cuda:0"


def _case(name, op, B, K, d_t, d_d, V, dtype="bf16", w="same", p_match=0.7, clf_b=0.0, tau=0.5, **more):
    return dict(name=name, op=op, B=B, K=K, d_t=d_t, d_d=d_d, V=V, dtype=dtype, w=w, p_match=p_match, clf_b=clf_b,
                tau=tau, **more)


def listed():
    return [
        # the smallest call: the fp32 workload of the benchmark's recipe; launches and latency are all there is
        _case("tiny_f32", "verify", 1, 8, 256, 128, 1024, "f32"),
        # fp32 storage at a small model's size (a 32k vocabulary), a few windows at once
        _case("f32_b4_k16", "verify", 4, 16, 2048, 1024, 32000, "f32"),
        # batch-1 decoding of an 8B-class target through the entry point that allocates nothing
        _case("static_8b_b1_k16", "static", 1, 16, 4096, 2048, 128256, p_match=0.8),
        # batch-1 decoding of a 70B-class target, the paper's window of 64
        _case("70b_b1_k64", "verify", 1, 64, 8192, 4096, 128256, clf_b=-1.0),
        # a server's small batch on a 70B-class target
        _case("70b_b8_k32", "verify", 8, 32, 8192, 4096, 128256, clf_b=-1.0),
        # a server's ordinary batch on an 8B-class target
        _case("8b_b32_k32", "verify", 32, 32, 4096, 2048, 128256, p_match=0.75),
        # the largest batch: 128 windows of 64 on a 70B-class target
        _case("70b_b128_k64", "verify", 128, 64, 8192, 4096, 128256, p_match=0.5, tau=0.6),
        # stochastic decoding (Gumbel-max) of a medium batch
        _case("sampled_8b_b12_k32", "sampled", 12, 32, 4096, 2048, 128256, inv_temperature=1.5),
        # the top-K baseline on a small batch
        _case("topk_8b_b8_k16", "topk", 8, 16, 4096, 0, 128256, top_k=8),
        # draft trees of 60 nodes, judge on target states only, a 32k vocabulary
        _case("tree_b2_k60", "tree", 2, 60, 4096, 0, 32000),
        # FP8 LM head, a few windows on a 70B-class target
        _case("fp8_70b_b3_k32", "verify", 3, 32, 8192, 4096, 128256, w="fp8", clf_b=-1.0),
        # ragged on every side: hidden sizes that are only multiples of 8, an odd vocabulary
        _case("ragged_b3_k20", "verify", 3, 20, 2888, 1000, 50257),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["verify", "verify", "verify", "static", "sampled", "topk", "tree"])
    storage = rng.choice(["bf16", "bf16", "bf16", "bf16", "fp8", "f32"])
    if op == "topk" and storage == "fp8":
        storage = "bf16"                        # the top-K baseline takes no FP8 weights
    # hidden sizes: mostly multiples of 256, as model families have them; some only of 128, 64 or 8
    g = {"fp8": 512, "f32": rng.choice([256, 4])}.get(storage) or rng.choice([256, 256, 256, 256, 128, 64, 8])
    d_t = max(1, round(_log_uniform(rng, 1024, 8192) / g)) * g
    d_d = rng.choice([0, d_t // 2 // 8 * 8])
    V = int(_log_uniform(rng, 16000, 152064))
    if rng.random() < 0.5:
        V = V // 64 * 64                        # vocabularies are often padded
    K = int(_log_uniform(rng, 3, 65))
    B = int(_log_uniform(rng, 1, 129))
    # keep a drawn case below the largest listed one: fp32 runs at a fraction of the bf16 rate, and hidden sizes that
    # are no multiple of 64 at less than the others
    most_flops = {"f32": 8e10, "fp8": 1e13}.get(storage) or (1.6e13 if d_t % 256 == 0 else 4e12 if d_t % 64 == 0 else 2e12)

    def fits(b):
        m = b * (K + 1)
        if 2.0 * m * V * d_t > most_flops or 4 * m > V:
            return False
        if storage == "fp8" and m > 272:
            return False
        return op != "static" or m * (-(-V // 64) * 8 + 12) + 2048 <= 8 << 20     # the static workspace, at its finest split

    while B > 1 and not fits(B):
        B = (B + 1) // 2
    while K > 1 and not fits(B):
        K = (K + 1) // 2
    more = {}
    if op == "sampled":
        more["inv_temperature"] = round(rng.uniform(0.7, 2.0), 2)
    if op == "topk":
        more["top_k"] = rng.choice([2, 4, 8, 16, 64])
        d_d = 0
    case = _case("", op, B, K, d_t, d_d, V, "f32" if storage == "f32" else "bf16", "fp8" if storage == "fp8" else "same",
                 p_match=round(rng.uniform(0.5, 0.9), 2), clf_b=rng.choice([0.0, -1.0]), tau=rng.choice([0.3, 0.5, 0.6]), **more)
    del case["name"]
    return case


class _Handle:
    """A library handle that goes away with the state that holds it."""

    def __init__(self, c):
        flags = aj.AJ_FLAG_TOPK if c["op"] == "topk" else 0
        self.h = aj.aj_create(c["B"], c["K"], c["d_t"], c["d_d"], c["V"], *_types(c)[:1], 1, flags, aj.AJ_KERNEL_AUTO,
                              _types(c)[1])

    def __del__(self):
        torch.cuda.synchronize()
        aj.aj_destroy(self.h)


class _DeviceArray:
    def __init__(self, address, n, typestr, owner):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": typestr, "data": (address, False), "version": 2}


def _types(c):
    return (aj.AJ_F32 if c["dtype"] == "f32" else aj.AJ_BF16), (aj.AJ_W_FP8_E4M3 if c["w"] == "fp8" else aj.AJ_W_SAME)


def prepare(c, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    B, K, d, V = c["B"], c["K"], c["d_t"], c["V"]
    M, D = B * (K + 1), c["d_t"] + c["d_d"]
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def normal(*shape, std=1.0, dtype=dt):
        return torch.randn(*shape, generator=g, device=DEVICE, dtype=dtype).mul_(std)

    def uniform(n, lo=0.0, hi=1.0):
        return torch.rand(n, generator=g, device=DEVICE) * (hi - lo) + lo

    def states(width):
        x = normal(M, width, dtype=torch.float32)
        return (x / x.square().mean(1, keepdim=True).sqrt()).to(dt)

    hidden_t = states(d)
    hidden_d = states(c["d_d"]) if c["d_d"] else None
    W = normal(V, d, std=0.02)
    clf_w = normal(D, std=1.0 / math.sqrt(D))

    # every row's favourite and second token, 6.5 .. 9 and 0.5 .. 1.5 less standard deviations of a logit
    tokens = torch.randperm(V, generator=g, device=DEVICE)
    tokens = tokens[torch.arange(2 * M, device=DEVICE) % V].view(2, M)
    first = uniform(M, 6.5, 9.0)
    level = torch.stack([first, first - uniform(M, 0.5, 1.5)]) * (0.02 * math.sqrt(d))
    h = hidden_t.float()
    for which in range(2):
        rows = W[tokens[which]].float()
        gain = (level[which] - (rows * h).sum(1)) / h.square().sum(1)
        W[tokens[which]] = (rows + gain[:, None] * h).to(dt)
    del h, rows

    slot = lambda x: x.view(B, K + 1)[:, :K]  # noqa: E731
    match = uniform(B * K).view(B, K) < c["p_match"]
    second = uniform(B * K).view(B, K) < 0.5
    other = torch.randint(0, V, (B, K), generator=g, device=DEVICE)
    draft = torch.where(match, slot(tokens[0]), torch.where(second, slot(tokens[1]), other)).to(torch.int32).contiguous()

    if c["w"] == "fp8":
        scale = W.abs().max().float() / 440.0
        W = torch.cat([(x.float() / scale).to(torch.float8_e4m3fn) for x in W.split(16384)]).view(torch.uint8)

    s = dict(case=c, hidden_t=hidden_t, hidden_d=hidden_d, W=W, clf_w=clf_w, draft=draft,
             out_len=torch.zeros(B, dtype=torch.int32, device=DEVICE), out_tok=torch.zeros(B, dtype=torch.int32, device=DEVICE))
    s["out"] = {"out_len": s["out_len"], "out_tok": s["out_tok"]}
    if c["op"] == "sampled":
        s["row_key"] = torch.randint(-2**62, 2**62, (B, K + 1), generator=g, device=DEVICE, dtype=torch.int64)
    if c["op"] == "tree":
        span = torch.arange(1, K + 1, device=DEVICE)            # node j hangs under one of -1 .. j-1
        s["parent"] = ((uniform(B * K).view(B, K) * span).long().clamp(max=span - 1) - 1).to(torch.int32).contiguous()
        s["out_node"] = s["out"]["out_node"] = torch.zeros(B, dtype=torch.int32, device=DEVICE)
    if c["op"] != "static":
        handle = s["handle"] = _Handle(c)
        t_star, maxlogit, _ = aj.aj_debug_ptrs(handle.h)
        # the greedy (or sampled) tokens and their logits, in the handle's own buffers
        s["out"]["t_star"] = torch.as_tensor(_DeviceArray(t_star, M, "<i4", handle), device=DEVICE)
        s["out"]["maxlogit"] = torch.as_tensor(_DeviceArray(maxlogit, M, "<f4", handle), device=DEVICE)
    return s


def run(s):
    c = s["case"]
    if c["op"] == "static":
        dtype, w_dtype = _types(c)
        aj.aj_verify_static(c["B"], c["K"], c["d_t"], c["d_d"], c["V"], dtype, 1, aj.AJ_KERNEL_AUTO, s["hidden_t"],
                            s["hidden_d"], s["W"], s["draft"], s["clf_w"], c["clf_b"], c["tau"], s["out_len"],
                            s["out_tok"], w_dtype=w_dtype)
        return s["out"]
    h = s["handle"].h
    if c["op"] == "verify":
        aj.aj_verify(h, s["hidden_t"], s["hidden_d"], s["W"], s["draft"], s["clf_w"], c["clf_b"], c["tau"],
                     s["out_len"], s["out_tok"])
    elif c["op"] == "sampled":
        aj.aj_verify_sampled(h, s["hidden_t"], s["hidden_d"], s["W"], s["draft"], s["clf_w"], c["clf_b"], c["tau"],
                             c["inv_temperature"], s["row_key"], s["out_len"], s["out_tok"])
    elif c["op"] == "tree":
        aj.aj_verify_tree(h, s["hidden_t"], s["hidden_d"], s["W"], s["draft"], s["parent"], s["clf_w"], c["clf_b"],
                          c["tau"], s["out_len"], s["out_tok"], s["out_node"])
    else:
        aj.aj_verify_topk(h, s["hidden_t"], s["W"], s["draft"], c["top_k"], s["out_len"], s["out_tok"])
    return s["out"]


def work(c):
    B, K, d, V = c["B"], c["K"], c["d_t"], c["V"]
    M, es = B * (K + 1), 4 if c["dtype"] == "f32" else 2
    judged = 0 if c["op"] == "topk" else B * K * (1.0 - c["p_match"])     # the judge looks at mismatching slots only
    small = B * K * 4 + B * 8 + M * 8 + (M * 8 if c["op"] == "sampled" else 0) + (B * K * 4 if c["op"] == "tree" else 0)
    return {"bytes": V * d * (1 if c["w"] == "fp8" else es) + M * d * es + judged * c["d_d"] * es + (d + c["d_d"]) * es + small,
            "flops": 2.0 * M * V * d + 2.0 * judged * (d + c["d_d"])}


def tolerance(c):
    # tokens, lengths and nodes are whole numbers, and the planted tokens keep every maximum apart.  The maxima are
    # sums of d_t products in fp32: against sums in fp64 the path is off by 2e-7 .. 7e-7 (2-norm) and by up to 1.7e-6
    # (largest difference) over the listed cases; four times that is allowed
    return {"rel": 2.8e-6, "max": 7e-6}
