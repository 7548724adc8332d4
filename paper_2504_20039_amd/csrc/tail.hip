// Steps 2 (second half) to 4: cross-block greedy maximum, mismatch test + judge, first-reject scan.
// Two forms.  k_verify_tail does everything in one launch with one workgroup per speculation window: right for
// short windows.  For few windows of many rows (batch 1 with 33 or 65 verify rows has ONE
// workgroup walk 65 rows x 1024 partials in five dependent rounds) the work is split by verify row instead:
// k_tail_rows gives every row a wave of its own (maximum of the row's partials, mismatch test of the row's slot,
// judge dot product at a mismatch), k_tail_scan then finds each window's first rejected slot.  In a draft tree a node is checked against its PARENT's row,
// which another wave reduces: there k_tail_rows judges every node, mismatch or not, and k_tree_scan tests the mismatches.
#include <stdlib.h>

#include "aj_internal.h"
#include "dot.h"

namespace aj {

namespace {

constexpr int TAIL_WAVES = 16;
constexpr int MAXK = 1023;

// Accepted node of greatest depth (lowest index among equals) of a draft tree of K <= blockDim.x nodes, by every thread of
// the workgroup: node j has parent p in [-1, j) and is rejected itself or not; it is accepted when no node on its path to
// the root is.  Pointer doubling: after i rounds a node knows whether one of its 2^i nearest (itself included) is
// rejected and where the rest of its path begins, so that K nodes take log2(K) rounds (a walk by one lane took K
// dependent steps: 60 nodes 20 us for the whole tail, 10 with this and the split form).  Returns depth << 16 | (0xffff - node), 0 if none.
// Up to 64 nodes one wave does it with shuffles, without a barrier (deepest_accepted_wave; with the workgroup's barriers trees of
// up to 8 nodes lost 0.2 .. 0.5 us against the walk by one lane, trees of 16 now gain 1).
__device__ __forceinline__ uint32_t deepest_accepted(int K, int p, bool rejected, int32_t *s_anc, int32_t *s_len, uint32_t *s_best)
{
    const int j = threadIdx.x;
    int anc = j < K ? p : -1, len = j < K && !rejected ? 1 : -(1 << 20);     // a rejected node makes every sum negative
    if (j == 0) *s_best = 0;
    if (j < K) {
        s_anc[j] = anc;
        s_len[j] = len;
    }
    __syncthreads();
    for (int span = 1; span < K; span <<= 1) {
        int na = -1, nl = 0;
        if (anc >= 0) {
            na = s_anc[anc];
            nl = s_len[anc];
        }
        __syncthreads();
        anc = na;
        len = max(len + nl, -(1 << 20));
        if (j < K) {
            s_anc[j] = anc;
            s_len[j] = len;
        }
        __syncthreads();
    }
    if (j < K && len > 0) atomicMax(s_best, (uint32_t)len << 16 | (uint32_t)(0xffff - j));
    __syncthreads();
    return *s_best;
}

__device__ __forceinline__ uint32_t deepest_accepted_wave(int K, int p, bool rejected, int lane)
{
    int anc = lane < K ? p : -1, len = lane < K && !rejected ? 1 : -(1 << 20);
    for (int span = 1; span < K; span <<= 1) {
        const int from = max(anc, 0), na = __shfl(anc, from), nl = __shfl(len, from);
        len = anc < 0 ? len : max(len + nl, -(1 << 20));
        anc = anc < 0 ? -1 : na;
    }
    uint32_t best = lane < K && len > 0 ? (uint32_t)len << 16 | (uint32_t)(0xffff - lane) : 0;
    for (int off = 1; off < K; off <<= 1) best = max(best, (uint32_t)__shfl_xor((int)best, off));     // nodes 0 .. K - 1: whole in lane 0
    return best;
}

// Phase 1: a wave per verify row reduces the row's block partials (coalesced: they are stored
//          [row][block]) with lowest-index tie-break.
// Phase 2: a wave per slot; at a mismatching slot (wave-uniform) its lanes share the judge dot
//          product and reduce it with cross-lane shuffles.
// Phase 3: wave 0 finds the first rejected slot with ballots and emits.
// TREE: the K slots are nodes of a draft tree (a.parent[b][j] in [-1, j)): node j is checked against the
//          greedy token of its parent's row, phase 3 finds the accepted node of greatest depth.
template <bool BF16, bool TREE>
__global__ __launch_bounds__(TAIL_WAVES * 64) void k_verify_tail(TailArgs a)
{
    __shared__ int32_t s_t[MAXK + 1];
    __shared__ uint8_t s_rej[MAXK + 1];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int K = a.K, R = K + 1;
    const size_t es = BF16 ? 2 : 4;
    // a thread's node's parent, for phase 3: requested before anything waits
    const int parent = TREE && (int)threadIdx.x < K ? a.parent[(size_t)b * K + threadIdx.x] : -1;

    for (int j = wave; j < R; j += TAIL_WAVES) {
        const size_t row = (size_t)b * R + j;
        const Best *p = a.part + row * a.nblocks;
        float bv = -INFINITY;
        int32_t bi = 0x7fffffff;
        for (int nb0 = lane; nb0 < a.nblocks; nb0 += 256) {       // 4 loads in flight per lane
            Best x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int nb = nb0 + 64 * u;
                x[u] = nb < a.nblocks ? p[nb] : Best{-INFINITY, 0x7fffffff};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (better(x[u].v, x[u].i, bv, bi)) {
                    bv = x[u].v;
                    bi = x[u].i;
                }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            float ov = __shfl_xor(bv, off);
            int32_t oi = __shfl_xor(bi, off);
            if (better(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
        }
        bi = row_token(bi);
        if (lane == 0) {
            s_t[j] = bi;
            a.t_star[row] = bi;
            a.maxlogit[row] = bv;
        }
    }
    __syncthreads();

    for (int j = wave; j < K; j += TAIL_WAVES) {
        // row whose prediction slot j is checked against: j in a chain, the parent's row in a tree
        // (a parent outside [-1, j) is clamped into it: malformed input stays inside the window's rows)
        const int prow = TREE ? min(max(a.parent[(size_t)b * K + j], -1), j - 1) + 1 : j;
        const bool mis = s_t[prow] != a.draft_tok[(size_t)b * K + j];
        float z = __builtin_nanf("");
        bool r = false;
        if (mis) {
            const size_t row = (size_t)b * R + (TREE ? (a.feat_offset ? j + 1 : prow) : j + a.feat_offset);
            // target half: from the LM-head pass (fused judge row), else a dot product here
            float acc = a.zt ? (lane == 0 ? a.zt[row] : 0.f)
                             : dot_part<BF16>((const char *)a.hidden_t + row * a.d_t * es, a.clf_w, a.d_t, lane);
            if (a.d_d > 0)
                acc += dot_part<BF16>((const char *)a.hidden_d + row * a.d_d * es,
                                      (const char *)a.clf_w + (size_t)a.d_t * es, a.d_d, lane);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            z = acc + a.clf_b;
            r = !(z < a.zthr);
        }
        if (lane == 0) {
            s_rej[j] = r;
            if (a.score) {
                a.score[(size_t)b * K + j] = z;
                a.score[(size_t)a.B * K + (size_t)b * K + j] = 1.f / (1.f + expf(-z));
            }
        }
    }
    __syncthreads();

    if (TREE) {
        __shared__ int32_t s_anc[MAXK], s_len[MAXK];
        __shared__ uint32_t s_best;
        const int j = threadIdx.x;
        if (K <= 64 && j >= 64) return;
        const int p = min(max(parent, -1), j - 1);
        const bool rejected = j < K && s_rej[j];
        const uint32_t best = K <= 64 ? deepest_accepted_wave(K, p, rejected, j) : deepest_accepted(K, p, rejected, s_anc, s_len, &s_best);
        if (threadIdx.x == 0) {
            const int node = best ? 0xffff - (int)(best & 0xffff) : -1;
            a.out_len[b] = (int)(best >> 16);
            a.out_tok[b] = s_t[node + 1];
            a.out_node[b] = node;
        }
        return;
    }
    if (wave == 0) {
        int n = K;
        for (int base = 0; base < K; base += 64) {
            const int j = base + lane;
            const bool r = j < K && s_rej[j];
            const unsigned long long m = __ballot(r);
            if (m) {
                n = base + __builtin_ctzll(m);
                break;
            }
        }
        if (lane == 0) {
            a.out_len[b] = n;
            a.out_tok[b] = s_t[n];
        }
    }
}

// Split form, first kernel: a wave per verify row (4 rows per workgroup).  All of a row's partials are requested
// before any is used (8 loads per lane in flight), so the row costs one memory round trip, the mismatch test a
// second (the draft token is requested with the partials) and a judge dot product two more.
constexpr int ROWS_PER_WG = 4;
template <bool BF16, bool TREE>
__global__ __launch_bounds__(ROWS_PER_WG * 64) void k_tail_rows(TailArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int K = a.K, R = K + 1;
    const int row = blockIdx.x * ROWS_PER_WG + wave;
    if (row >= a.B * R) return;
    const int b = row / R, j = row - b * R;
    const size_t es = BF16 ? 2 : 4;
    const int32_t dtok = !TREE && j < K ? a.draft_tok[(size_t)b * K + j] : 0;

    const Best *p = a.part + (size_t)row * a.nblocks;
    float bv = -INFINITY;
    int32_t bi = 0x7fffffff;
    constexpr int U = 8;
    for (int nb0 = lane; nb0 < a.nblocks; nb0 += 64 * U) {
        Best x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int nb = nb0 + 64 * u;
            x[u] = nb < a.nblocks ? p[nb] : Best{-INFINITY, 0x7fffffff};
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (better(x[u].v, x[u].i, bv, bi)) {
                bv = x[u].v;
                bi = x[u].i;
            }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        float ov = __shfl_xor(bv, off);
        int32_t oi = __shfl_xor(bi, off);
        if (better(ov, oi, bv, bi)) {
            bv = ov;
            bi = oi;
        }
    }
    bi = row_token(bi);
    if (lane == 0) {
        a.t_star[row] = bi;
        a.maxlogit[row] = bv;
    }
    // a chain's row j: slot j, judged at a mismatch only.  A tree's row j: node j - 1, judged whether it matches or not
    const int slot = TREE ? j - 1 : j;
    if (TREE ? slot < 0 : slot >= K) return;

    const bool mis = TREE || bi != dtok;    // wave-uniform: every lane holds the reduced maximum
    float z = __builtin_nanf("");
    bool r = false;
    if (mis) {
        // chain: same window, j + feat_offset <= K; tree: the node's own row or its parent's
        const size_t frow = !TREE ? (size_t)row + a.feat_offset
                                  : a.feat_offset ? (size_t)row
                                                  : (size_t)b * R + min(max(a.parent[(size_t)b * K + slot], -1), slot - 1) + 1;
        float acc = a.zt ? (lane == 0 ? a.zt[frow] : 0.f)
                         : dot_part<BF16, 8>((const char *)a.hidden_t + frow * a.d_t * es, a.clf_w, a.d_t, lane);
        if (a.d_d > 0)
            acc += dot_part<BF16, 8>((const char *)a.hidden_d + frow * a.d_d * es,
                                     (const char *)a.clf_w + (size_t)a.d_t * es, a.d_d, lane);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        z = acc + a.clf_b;
        r = !(z < a.zthr);
    }
    if (lane == 0) {
        a.rej[(size_t)b * K + slot] = r;
        if (a.score) {
            a.score[(size_t)b * K + slot] = z;
            a.score[(size_t)a.B * K + (size_t)b * K + slot] = 1.f / (1.f + expf(-z));
        }
    }
}

// Split form of a draft tree, second kernel: a workgroup per window, a thread per node.
__global__ __launch_bounds__(1024) void k_tree_scan(TailArgs a)
{
    __shared__ int32_t s_anc[MAXK], s_len[MAXK];
    __shared__ uint32_t s_best;
    const int b = blockIdx.x, j = threadIdx.x, K = a.K;
    const size_t row0 = (size_t)b * (K + 1), slot = (size_t)b * K + j;
    int p = -1;
    bool rejected = false;
    if (j < K) {
        p = min(max(a.parent[slot], -1), j - 1);
        const bool mis = a.t_star[row0 + p + 1] != a.draft_tok[slot];
        rejected = mis && a.rej[slot];
        if (a.score && !mis) a.score[slot] = a.score[(size_t)a.B * K + slot] = __builtin_nanf("");    // not judged
    }
    const uint32_t best = K <= 64 ? deepest_accepted_wave(K, p, rejected, j) : deepest_accepted(K, p, rejected, s_anc, s_len, &s_best);
    if (j == 0) {
        const int node = best ? 0xffff - (int)(best & 0xffff) : -1;
        a.out_len[b] = (int)(best >> 16);
        a.out_tok[b] = a.t_star[row0 + node + 1];
        a.out_node[b] = node;
    }
}

// Split form, second kernel: a wave per window finds the first rejected slot with ballots and emits.
__global__ __launch_bounds__(64) void k_tail_scan(TailArgs a)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const int K = a.K;
    int n = K;
    for (int base = 0; base < K; base += 64) {
        const int j = base + lane;
        const bool r = j < K && a.rej[(size_t)b * K + j];
        const unsigned long long m = __ballot(r);
        if (m) {
            n = base + __builtin_ctzll(m);
            break;
        }
    }
    if (lane == 0) {
        a.out_len[b] = n;
        a.out_tok[b] = a.t_star[(size_t)b * (K + 1) + n];
    }
}

constexpr int SPLIT_TREE = 28;      // nodes of a draft tree from which the split form pays

// 1: split form, 0: one launch; AJ_TAIL=split|fused in the environment overrides the choice (for measurements)
bool use_split_tail(const TailArgs &a)
{
    static const int forced = [] {
        const char *e = getenv("AJ_TAIL");
        return !e ? -1 : (e[0] == 's' ? 1 : (e[0] == 'f' ? 0 : -1));
    }();
    if (!a.rej) return false;
    if (forced >= 0) return forced == 1;
    // Trees: a window's nodes take a workgroup several rounds; the split form spreads them over the chip but judges every node
    // instead of the mismatching ones, so it pays later the more tokens match.  Whole calls, one launch with the walk by one lane
    // -> split, us, half / 0.95 of the tokens matching, 4096 + 2048 features: 1 x 24 nodes -2.0 / +0.7 (one launch with the wave's scan:
    // -1.5 / -1.5), 1 x 28 -3.4 / -1.0, 32 x 28 -4.2 / -2.4, 1 x 63 x 256 -9 / -6; above 1024 rows (25 MB of features at 8192 + 4096)
    // the extra reads cost more
    if (a.parent) return a.K >= SPLIT_TREE && a.B * (a.K + 1) <= 1024;
    // Chains.  Windows of up to 13 rows (16 waves take them in one round), and a few of up to 17, are cheaper in one launch up to 512
    // of them: whole calls, split -> one launch, us, 4096 + 2048 features: 8 x 5 rows 50.9 -> 48.9, 16 x 9 84.9 -> 82.8, 64 x 9 x 2048 76.4 ->
    // 74.1, 128 x 9 246.8 -> 244.5, 4 x 17 55.1 -> 54.5 (2048 + 1024: 34.4 -> 33.1), but 32 x 17 at 8192 + 4096 240 -> 248.  Longer windows: the split form
    // wins from 33 rows on (6 against 16 us at 1 x 33 rows, 11 against 27 at 1 x 65, 13 against 26 at 8 x 33, 15 against 51 at 128 x
    // 65); at 17 rows the one launch is a microsecond cheaper
    // Beyond 512 windows a launch of 16-wave workgroups takes several rounds: 700 x 5 x 2048 + 1024 as fast either way, 2000 x 3 x 4096 1188 -> 1198
    if ((a.K <= 12 && a.B <= 512) || (a.K <= 16 && a.B <= 4)) return false;
    return a.B * (a.K + 1) > 32;
}

}  // namespace

hipError_t verify_tail(const TailArgs &a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (use_split_tail(a)) {
        const int rows = a.B * (a.K + 1);
        const int grid = (rows + ROWS_PER_WG - 1) / ROWS_PER_WG;
        const dim3 block(ROWS_PER_WG * 64);
        if (a.parent) {
            if (a.dtype == 1) hipLaunchKernelGGL((k_tail_rows<true, true>), dim3(grid), block, 0, s, a);
            else hipLaunchKernelGGL((k_tail_rows<false, true>), dim3(grid), block, 0, s, a);
        } else {
            if (a.dtype == 1) hipLaunchKernelGGL((k_tail_rows<true, false>), dim3(grid), block, 0, s, a);
            else hipLaunchKernelGGL((k_tail_rows<false, false>), dim3(grid), block, 0, s, a);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (a.parent) hipLaunchKernelGGL(k_tree_scan, dim3(a.B), dim3((a.K + 63) / 64 * 64), 0, s, a);
        else hipLaunchKernelGGL(k_tail_scan, dim3(a.B), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    if (a.parent) {
        if (a.dtype == 1) hipLaunchKernelGGL((k_verify_tail<true, true>), dim3(a.B), dim3(TAIL_WAVES * 64), 0, s, a);
        else hipLaunchKernelGGL((k_verify_tail<false, true>), dim3(a.B), dim3(TAIL_WAVES * 64), 0, s, a);
    } else {
        if (a.dtype == 1) hipLaunchKernelGGL((k_verify_tail<true, false>), dim3(a.B), dim3(TAIL_WAVES * 64), 0, s, a);
        else hipLaunchKernelGGL((k_verify_tail<false, false>), dim3(a.B), dim3(TAIL_WAVES * 64), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace aj
