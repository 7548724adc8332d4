// LM head + per-block greedy maximum for fp32 storage, on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: the
// products and sums are IEEE fp32, as with plain FMAs).
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s nominal, 134 reached by a large library product here) from about
// 30 verify rows on, HBM below.  An fp32 MFMA runs for 32 cycles on 2 x 64 operand floats, so the operands need no LDS:
// a wave loads both straight into registers in MFMA layout.  The k order of a sum is free, so a lane takes FOUR
// consecutive k elements per 16-byte load (element e feeds MFMA e) and two loads cover whole
// 128-byte lines of 16 rows.
//   * A wave holds NB x MB blocks of 16 vocabulary rows x 16 verify rows; one step of 32 k elements is 8 NB MB MFMAs
//     (5120 cycles at 4 x 5) over 2 (NB + MB) loads, issued one step ahead: the L2 -> CU traffic of the largest tile is
//     14 B per cycle and compute unit, far below what the path moves.
//   * The 4 waves of a workgroup split k, because a model's vocabulary is only V / 64 tiles (500 at V = 32000: not two
//     waves per SIMD); their partial blocks meet in LDS once, at the end.  Some problems take fewer vocabulary blocks
//     per tile (NB = 3, 2, 1), so that all compute units have work: see choose().
// Measured (kernel and tail, us): 68 rows x 2048 x 32000 671 -> 104 against plain FMAs on LDS tiles of 64 x 16, 17 rows x
// 2048 x 107552 788 -> 172 (5.1 TB/s), 816 rows x 2304 x 19996 3308 -> 667 (113 TFLOP/s), 9 rows x 256 x 1024 25 -> 11.
#include <type_traits>

#include "../../include/aj.h"
#include "aj_internal.h"

namespace aj {

namespace {

constexpr int FWAVES = 4;
constexpr int FSTEP = 32;            // k elements per step: one 128-byte line of every row
// Longest row whose offsets within the largest tile, up to 80 rows of 4 d bytes, stay below 2^32.  Longer rows take one tile
// (1 x 4 blocks) with 64-bit offsets
constexpr int LONG_ROW = 1 << 23;

template <int MB, int NB, bool NT, bool DUMP, bool LONG = false>
__global__ __launch_bounds__(FWAVES * 64, !LONG && MB * NB * 4 + (MB + NB) * 16 <= 104 ? 4 : 2) void k_lm_head_f32(LmHeadArgs a)
{
    static_assert((uint64_t)(16 * (MB > NB ? MB : NB)) * LONG_ROW * 4 < 1ull << 32, "32-bit byte offsets within a tile");
    using offset_t = typename std::conditional<LONG, uint64_t, uint32_t>::type;
    constexpr int NP = NB * MB;                                   // accumulator blocks of a wave
    __shared__ f32x4 xch[NP][FWAVES - 1][64];                     // partial blocks, by block, source and lane
    __shared__ Best red[NB][MB * 16];
    __shared__ int32_t redc[NB][MB * 16];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    // the row tiles of a vocabulary tile go to consecutive workgroups of one XCD (id mod 8; gridDim.x is a multiple of 8),
    // which share its W_lm rows in L2.  Fewer than 8 vocabulary tiles would use as many XCDs: their row tiles go round all of
    // them (16000 rows x 64 x 64, whole call: 47 -> 22 us)
    const bool few = a.nblocks < 8;
    const int vt = few ? blockIdx.x % a.nblocks : blockIdx.y * 8 + (blockIdx.x & 7);
    const int mt = few ? blockIdx.x / a.nblocks : blockIdx.x >> 3;
    if (vt >= a.nblocks) return;
    const int v0 = vt * 16 * NB, m0 = mt * 16 * MB;
    const int d = a.d;
    const char *W = (const char *)a.W + (size_t)v0 * d * 4, *H = (const char *)a.H + (size_t)m0 * d * 4;
    offset_t wo[NB][2], ho[MB];         // row offsets; rows beyond the end repeat the last one (their logits are never looked at)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) wo[b][h] = (offset_t)min(b * 16 + h * 8 + (l16 & 7), a.V - 1 - v0) * (uint32_t)d * 4u;
#pragma unroll
    for (int y = 0; y < MB; ++y) ho[y] = (offset_t)min(y * 16 + l16, a.M - 1 - m0) * (uint32_t)d * 4u;

    const int nsteps = (d + FSTEP - 1) / FSTEP;
    const int s0 = nsteps * wave / FWAVES, s1 = nsteps * (wave + 1) / FWAVES;
    // where a wave's quarter is a multiple of 4096 bytes (other quarters start in different halves of them anyway)
    const bool weave = !LONG && (d & 4095) == 0;

    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int y = 0; y < MB; ++y) acc[b][y] = f32x4{0.f, 0.f, 0.f, 0.f};

    f32x4 fw[2][NB][2], fh[2][MB][2];
    // hidden_t: the lane's two 4-element groups of step s, k = 32 s + 16 c + 4 q4.  W_lm: load h of a block covers rows
    // 8h .. 8h+7 x the whole 128-byte line - lane (l16, q4) asks for row l16 % 8, bytes 64 (l16 / 8) + 16 q4 - because
    // whole lines stream faster than 16 rows x 64 B (0.9 GB of W_lm at 17 rows: 213 us, with whole non-temporal lines 172);
    // one DPP rotation by 8 lanes per register then gives group c of all 16 rows (see group()).  A group beyond d reads the row's last one instead.
    auto load = [&](int at, int set) {
        const int s = weave ? interleave_4k<32>(at) : at;
        const offset_t kw = (offset_t)min(s * FSTEP + (l16 >> 3) * 16 + q4 * 4, d - 4) * 4u;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 *p = (const f32x4 *)(W + (wo[b][h] + kw));
                fw[set][b][h] = NT ? __builtin_nontemporal_load(p) : *p;
            }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const offset_t kb = (offset_t)min(s * FSTEP + c * 16 + q4 * 4, d - 4) * 4u;
#pragma unroll
            for (int y = 0; y < MB; ++y) fh[set][y][c] = *(const f32x4 *)(H + (ho[y] + kb));
        }
    };
    // group c of the 16 rows of a block from its two loads: lane l16 <-> row l16
    auto group = [&](const f32x4 &x, const f32x4 &y, int c) {
        f32x4 r;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int xi = __float_as_int(x[k]), yi = __float_as_int(y[k]);
            r[k] = __int_as_float(c == 0 ? __builtin_amdgcn_update_dpp(xi, yi, 0x128 /* row_ror:8 */, 0xF, 0xC, false)
                                         : __builtin_amdgcn_update_dpp(yi, xi, 0x128, 0xF, 0x3, false));
        }
        return r;
    };
    auto compute = [&](int s, int set) {
        // blocks whose MFMAs interleave: with few verify rows all of them (an MFMA waits for the one before it on the same
        // accumulator), else one at a time, which saves the registers of the others' rotated operands
        constexpr int NI = MB <= 3 ? NB : 1;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b0 = 0; b0 < NB; b0 += NI) {
                f32x4 w[NI];
#pragma unroll
                for (int b = 0; b < NI; ++b) w[b] = group(fw[set][b0 + b][0], fw[set][b0 + b][1], c);
                if ((s + 1) * FSTEP > d && s * FSTEP + c * 16 + q4 * 4 >= d) {     // the row's ragged end counts as zero
#pragma unroll
                    for (int b = 0; b < NI; ++b) w[b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < NI; ++b)
#pragma unroll
                        for (int y = 0; y < MB; ++y)
                            acc[b0 + b][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[b][e], fh[set][y][c][e], acc[b0 + b][y], 0, 0, 0);
            }
    };
    if (s0 < s1) load(s0, 0);
    int s = s0;
    for (; s + 1 < s1; s += 2) {
        load(s + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        compute(s, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(min(s + 2, s1 - 1), 0);
        __builtin_amdgcn_sched_barrier(0);
        compute(s + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (s < s1) compute(s, 0);

    // ---- the 4 k parts of a block meet in its owner, wave (block mod 4), summed in ascending wave order
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int own = p & 3;
        if (wave != own) xch[p][wave < own ? wave : wave - 1][lane] = acc[p / MB][p % MB];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int own = p & 3, b = p / MB, y = p % MB;
        if (wave != own) continue;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < FWAVES; ++w) sum += w == own ? acc[b][y] : xch[p][w < own ? w : w - 1][lane];
        // lane (l16, q4): verify row 16 y + l16 against vocabulary rows 16 b + 4 q4 + r, ascending in r
        const int row = m0 + y * 16 + l16, rowc = min(row, a.M - 1);
        float th = INFINITY;
        int32_t tk = -1;
        if (a.thr) {                 // top-K baseline: the row's draft token
            th = a.thr[rowc];
            tk = a.thr_tok[rowc];
        }
        uint32_t klo = 0, khi = 0;
        if (a.key) {                 // sampling mode: the row's noise key
            klo = (uint32_t)a.key[rowc];
            khi = (uint32_t)(a.key[rowc] >> 32);
        }
        float bv = -INFINITY;
        int32_t bi = 0x7fffffff, cn = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int v = v0 + b * 16 + q4 * 4 + r;
            float val = sum[r];
            if (v < a.V) {
                if (DUMP && row < a.M) a.dump[(size_t)row * a.V + v] = val;
                if (a.key) val = fmaf(val, a.inv_temp, gumbel_noise(klo, khi, (uint32_t)v));
                if (val > bv) {
                    bv = val;
                    bi = v;
                }
                cn += ranks_before(val, v, th, tk);
            }
        }
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float ov = __shfl_xor(bv, off);
            const int32_t oi = __shfl_xor(bi, off);
            if (better(ov, oi, bv, bi)) {
                bv = ov;
                bi = oi;
            }
            cn += __shfl_xor(cn, off);
        }
        if (q4 == 0) {
            red[b][y * 16 + l16] = Best{bv, bi};
            redc[b][y * 16 + l16] = cn;
        }
    }
    __syncthreads();
    const int lr = threadIdx.x;
    if (lr < MB * 16 && m0 + lr < a.M) {
        Best best = red[0][lr];
        int32_t cn = redc[0][lr];
#pragma unroll
        for (int b = 1; b < NB; ++b) {
            if (better(red[b][lr].v, red[b][lr].i, best.v, best.i)) best = red[b][lr];
            cn += redc[b][lr];
        }
        a.part[(size_t)(m0 + lr) * a.nblocks + vt] = best;
        if (a.cnt) a.cnt[(size_t)(m0 + lr) * a.nblocks + vt] = cn;
    }
}

// Tile of M rows: the number of 16-row blocks per tile (at most 5: 4 x 5 accumulator blocks and two steps of operands
// fill the registers of two waves per SIMD) that pads least, and the number of vocabulary blocks per tile for which the
// busiest compute unit has least to do.  A tile of 3, 2 or 1 blocks loads more hidden_t per MFMA: 1.06, 1.17 and 1.8 times the
// time per block (57 rows x 6656 x 142208: 1056 / 1090 / 1368 us with 4 / 3 / 2; 68 rows x 2048 x 32000: 108 / 127 / 194 with
// 4 / 2 / 1), so it pays where it fills the last round of tiles better: 57 rows x 6656 x 36224 has 567 tiles of 4, 755 of 3 and
// 1132 of 2 for 256 compute units: 351 / 289 / 386 us in one run (289 .. 305 with the 3 over several); V = 17000: 235 / 191 / 232.
struct F32Tile {
    int mb, nb;
    double cost;        // rounds of tiles over the compute units x vocabulary blocks x their relative time
};
F32Tile choose(int M, int V, int d, int num_cus)
{
    if (d > LONG_ROW) return {1, 4, 0.0};
    const int blocks = (M + 15) / 16;
    int mb = blocks < 5 ? blocks : 5;
    if (blocks > 5)
        for (int c = 4; c >= 3; --c)
            if ((blocks + c - 1) / c * c < (blocks + mb - 1) / mb * mb) mb = c;
    const int64_t tm = (blocks + mb - 1) / mb;
    int nb = 4;
    double best = 0.0;
    for (int c = 4; c >= 1; --c) {
        const int64_t nblocks = (V + 16 * c - 1) / (16 * c), tiles = tm * nblocks;
        // smaller tiles mean more partials per row: never more than the static entry point has room for (large tiles of a
        // large problem need more anyway, and win there: see the rounds above)
        if (c < 4 && (uint64_t)M * nblocks * sizeof(Best) + 12ull * M + 1024 > AJ_STATIC_SCRATCH_BYTES) continue;
        const double cost = (double)((tiles + num_cus - 1) / num_cus) * c * (c == 4 ? 1.0 : c == 3 ? 1.06 : c == 2 ? 1.17 : 1.8);
        if (c == 4 || cost < best) {
            best = cost;
            nb = c;
        }
    }
    return {mb, nb, best};
}

dim3 grid_of(const LmHeadArgs &a, int tm)
{
    return dim3((unsigned)((a.nblocks < 8 ? a.nblocks : 8) * tm), (unsigned)((a.nblocks + 7) / 8));
}

template <int MB, int NB>
hipError_t launch(const LmHeadArgs &a, hipStream_t s)
{
    const int tm = (a.M + MB * 16 - 1) / (MB * 16);
    const dim3 grid = grid_of(a, tm);
    // W_lm is read once when there is one row tile: non-temporal, unless rows start inside a line, whose two parts then come
    // by different loads (57 rows x 4012 x 80832: 466 us non-temporal, 431 without; 2 rows 338, 255; whole lines, d = 6656: 610, 653)
    if (a.dump) hipLaunchKernelGGL((k_lm_head_f32<MB, NB, false, true>), grid, dim3(FWAVES * 64), 0, s, a);
    else if (tm == 1 && a.d % FSTEP == 0) hipLaunchKernelGGL((k_lm_head_f32<MB, NB, true, false>), grid, dim3(FWAVES * 64), 0, s, a);
    else hipLaunchKernelGGL((k_lm_head_f32<MB, NB, false, false>), grid, dim3(FWAVES * 64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_long(const LmHeadArgs &a, hipStream_t s)
{
    const dim3 grid = grid_of(a, (a.M + 15) / 16);
    if (a.dump) hipLaunchKernelGGL((k_lm_head_f32<1, 4, false, true, true>), grid, dim3(FWAVES * 64), 0, s, a);
    else hipLaunchKernelGGL((k_lm_head_f32<1, 4, false, false, true>), grid, dim3(FWAVES * 64), 0, s, a);
    return hipGetLastError();
}

template <int MB>
hipError_t launch_nb(const LmHeadArgs &a, int nb, hipStream_t s)
{
    return nb == 4 ? launch<MB, 4>(a, s) : nb == 3 ? launch<MB, 3>(a, s) : nb == 2 ? launch<MB, 2>(a, s) : launch<MB, 1>(a, s);
}

}  // namespace

int lm_head_f32_blocks(int M, int V, int d, int num_cus)
{
    if (M <= 0) return 1;
    const int nb = choose(M, V, d, num_cus).nb;
    return (V + 16 * nb - 1) / (16 * nb);
}

// fitted to 33 .. 1000 rows, d_t 1024 .. 8192, V 4096 .. 152064 (6 %), less launches and tail
double lm_head_f32_cost(int M, int V, int d, int num_cus)
{
    const F32Tile t = choose(M, V, d, num_cus);
    const double rounds = t.cost / (t.nb * (t.nb == 4 ? 1.0 : t.nb == 3 ? 1.06 : t.nb == 2 ? 1.17 : 1.8));
    const double matrix = t.cost * (1.04 * t.mb + 0.26) * d / 1000.0, stream = (double)V * d * 4 / 6e6;
    return 5.5 + 1.3 * rounds + (matrix > stream ? matrix : stream);
}

void lm_head_f32_tile(int M, int V, int d, int num_cus, int32_t *vocab_rows, int32_t *verify_rows)
{
    const F32Tile t = choose(M, V, d, num_cus);
    *vocab_rows = 16 * t.nb;
    *verify_rows = 16 * t.mb;
}

hipError_t lm_head_f32(const LmHeadArgs &a, int num_cus, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    if (a.d > LONG_ROW) return launch_long(a, s);
    const F32Tile t = choose(a.M, a.V, a.d, num_cus);
    switch (t.mb) {
        case 1: return launch_nb<1>(a, t.nb, s);
        case 2: return launch_nb<2>(a, t.nb, s);
        case 3: return launch_nb<3>(a, t.nb, s);
        case 4: return launch_nb<4>(a, t.nb, s);
        default: return launch_nb<5>(a, t.nb, s);
    }
}

}  // namespace aj
