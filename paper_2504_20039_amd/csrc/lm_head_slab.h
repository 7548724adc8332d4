// LM head (step 1) + per-vocabulary-block greedy maximum (first half of step 2): small workgroup tiles for shapes that
// leave the chip idle in the kernels with one large tile per compute unit (a vocabulary of 17000 is 34 workgroups of the
// accumulator-resident kernel, 67 of the wide one), and for hidden sizes that are no multiple of 64 or 32.
//
// What bounds it: the W_lm stream of a compute unit, at most 25 GB/s, so what counts is that all of them have the same share of the
// vocabulary, and that enough waves wait for it.
//   * A workgroup takes up to 64 NB vocabulary rows (NB 1 .. 4) x 16 MB verify rows, NB chosen for the shape.  Its height is not a
//     multiple of 16: each wave owns `rows` vocabulary rows, chosen so that the workgroups fill the compute units evenly, and the rows
//     of its last block beyond them lie outside its buffer, cost no traffic and are dropped at the end (24 rows x 7168 x 17000, 133
//     tiles of 128 rows -> 250 of 68: 61.5 -> 44.4 us; 63 x 2888 x 50257, 197 of 256 -> 252 of 200: 78.6 -> 70.2; deeper rings of W_lm,
//     3 or 4 slabs, gained nothing at either).
//   * One round of tiles (a workgroup per compute unit): 8, 12 or 16 waves of one block each (8 of two where 16 would have too few
//     registers): one's loads, LDS reads and barriers run behind the others' MFMAs (122 x 4096 x 32000 64.6 -> 61.0, 80 x 7168 x
//     36000 104 -> 94, 63 x 2888 x 50257 70.2 -> 65.4; FP8 99 x 7168 x 36000 0.77 of the time).  More rounds: 4 waves of NB blocks, two
//     workgroups per compute unit, which do the same for each other and read each hidden_t fragment from LDS less often (264 x 4096 x 100000:
//     12 waves take 1.1 times as long).  FP8 with one or two row blocks: 4 waves, the waves' own work being half.
//   * W_lm lines go global -> registers (whole 128-byte lines of 8 rows per load,
//     one DPP rotation per register to the MFMA layout, as in lm_head_resident.hip), a slab of 2 .. 8 loads ahead.
//   * hidden_t slabs are shared by the waves through LDS, double buffered, one barrier per slab; requested a slab ahead
//     into registers and written to LDS a slab later, so that the compiler counts every load itself.
//   * Both operands are buffer loads: rows beyond the wave's or beyond M and k elements beyond d_t lie outside the buffer and read as
//     zero, so any d_t that is a multiple of 8 takes the same loop.
// Measured (whole call, us; before the small tiles / tiles of full height and 4 waves / now): 24 rows x 7168 x 17000 208 / 67 / 52, 64 x 4096 x
// 32000 131 / 56 / 54, 122 x 4096 x 32000 93 / 73 / 70 (4.3 TB/s), 122 x 7168 x 72000 302 / 253 / 230, 264 x 7168 x 17000 182 / 152 / 121, 60 x 2888 x 50257
// 123 / 86 / 73, 99 x 7168 x 36000 - / 133 / 108, 500 x 2888 x 100000 660 / 427 / 427 (675 TFLOP/s); FP8 64 x 7168 x 32000 127 / 64 / 60, 99 x 7168 x
// 36000 - / 108 / 82.
#pragma once
#include "../../include/aj.h"
#include "aj_internal.h"

namespace aj {


// EVEN: the interleaved order of slabs (rows of a multiple of 4096 bytes).  A constant: chosen at run time it takes 18 registers more, which the
// largest tiles of 4 waves do not have (245 rows x 1552 x 61134: 139 us with the spills in the loop, 101 without)
template <int SL_WAVES, int MB, int NB, bool FP8W, bool NT, bool EVEN>
__global__ __launch_bounds__(SL_WAVES * 64, SL_WAVES == 4 ? 2 : SL_WAVES / 4) void k_lm_head_slab(LmHeadArgs a, int wrows, int rot_step)
{
    // 128-byte lines of a W_lm row per slab
    constexpr int LPS = FP8W ? (SL_WAVES * NB == 4 ? 2 : 1) : SL_WAVES == 4 ? 4 / NB : 2;
    constexpr int HLINE = FP8W ? 256 : 128;                      // bytes of a hidden_t row that meet one line of W_lm
    constexpr int HROW = HLINE * LPS;                            // ... and one slab
    constexpr int ROWS = MB * 16, HBUF = ROWS * HROW;
    constexpr int CPR = HROW / 16;                               // 16-byte chunks of a row per slab
    constexpr int NT_ = SL_WAVES * 64;
    constexpr int HCH = (ROWS * CPR + NT_ - 1) / NT_;            // chunks staged per thread and slab
    constexpr int KPH = FP8W ? 2 : 1;                            // k steps per half line
    constexpr int PPL = 2 * KPH, NP = LPS * PPL;                 // pieces (k steps of 32) per line, per slab
    constexpr uint32_t OUT = 0x80000000u;                        // a byte offset beyond every buffer: reads as zero
    __shared__ __attribute__((aligned(1024))) char lds[2 * HBUF];
    __shared__ Best red[SL_WAVES][ROWS];
    __shared__ int32_t redc[SL_WAVES][ROWS];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    // the row tiles of a vocabulary tile go to consecutive workgroups of one XCD (id mod 8; gridDim.x is a multiple of 8)
    const int vt = blockIdx.y * 8 + (blockIdx.x & 7), mt = blockIdx.x >> 3;
    if (vt >= a.nblocks) return;
    const int vw = (vt * SL_WAVES + wave) * wrows, m0 = mt * ROWS;       // first vocabulary row of the wave
    const int ve = min(vw + wrows, a.V);                                 // ... and the one after its last
    const uint32_t wrow = (uint32_t)a.d * (FP8W ? 1u : 2u), hrow = (uint32_t)a.d * 2u;
    // rows beyond V and M and k elements beyond d lie outside the buffers: they read as zero, without traffic
    auto buffer_of = [](const void *base, uint32_t bytes) {      // in scalar registers
        const uint64_t p = (uint64_t)base;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
        return __builtin_amdgcn_make_buffer_rsrc((void *)((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes),
                                                 0x00020000);
    };
    const auto wres = buffer_of((const char *)a.W + (size_t)min(vw, a.V - 1) * wrow,
                                (uint32_t)max(ve - vw, 0) * wrow);
    const auto hres = buffer_of((const char *)a.H + (size_t)m0 * hrow, (uint32_t)min(a.M - m0, ROWS) * hrow);

    const int NS = (int)((wrow + LPS * 128 - 1) / (LPS * 128));  // slabs
    const int rot = EVEN ? 0 : (int)((unsigned)(vt * rot_step) % (unsigned)NS);
    // byte offset, in rows of `bytes` per slab, of the slab of iteration `it`; beyond the last one OUT
    auto slab_of = [&](int it, int bytes) {
        const int s = EVEN ? interleave_4k<4096 / (LPS * 128)>(it) : it + rot;
        const uint32_t o = (uint32_t)(s >= NS ? s - NS : s) * (uint32_t)bytes;
        return it < NS ? o : OUT;
    };

    const uint32_t lanek = (uint32_t)(q4 + 4 * (l16 >> 3)) * 16u, wo = (uint32_t)(l16 & 7) * wrow;
    constexpr int HRS = NT_ / CPR;                               // hidden_t rows staged at a time
    const int hr0 = tid / CPR, hc0 = tid % CPR;
    const uint32_t ho = (uint32_t)hr0 * hrow;

    u32x4 ring[2][LPS][NB][2];
    auto load_w = [&](int it, int set, int l) {
        const uint32_t kb = slab_of(it, LPS * 128) + l * 128 + lanek;
        const uint32_t kk = kb < wrow ? kb : OUT;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                ring[set][l][b][h] = __builtin_amdgcn_raw_buffer_load_b128(wres, (int)(wo + kk + (uint32_t)(b * 16 + h * 8) * wrow), 0,
                                                                        NT ? 2 : 0);
    };
    u32x4 hst[HCH];
    auto load_h = [&](int it) {
        const uint32_t kb = slab_of(it, HROW) + (uint32_t)hc0 * 16u;
        const uint32_t kk = kb < hrow ? kb : OUT;
#pragma unroll
        for (int i = 0; i < HCH; ++i)
            if ((i + 1) * NT_ <= ROWS * CPR || tid + i * NT_ < ROWS * CPR)
                hst[i] = __builtin_amdgcn_raw_buffer_load_b128(hres, (int)(ho + kk + (uint32_t)(i * HRS) * hrow), 0, 0);
    };
    // chunk c of row r sits at chunk c ^ swz(r): the 16 rows a fragment read touches fall into different banks
    auto swz = [](int r) { return CPR == 8 ? (r >> 1) & 7 : r & 15; };
    static_assert(CPR == 8 ? HRS / 2 % 8 == 0 : CPR == 32 ? HRS % 8 == 0 : HRS % 16 == 0, "swz of the rows staged by a thread");
    const int hs0 = hr0 * HROW + ((hc0 ^ swz(hr0)) * 16), hs1 = HRS % 16 == 8 ? hr0 * HROW + ((hc0 ^ swz(hr0) ^ 8) * 16) : hs0;
    auto store_h = [&](int buf) {
#pragma unroll
        for (int i = 0; i < HCH; ++i)
            if ((i + 1) * NT_ <= ROWS * CPR || tid + i * NT_ < ROWS * CPR)
                *(u32x4 *)(lds + buf * HBUF + (i & 1 ? hs1 : hs0) + i * HRS * HROW) = hst[i];
    };
    // fragment of row block y for piece p: k elements of lane group q4 are those of its 16 bytes of the half line
    const int sw = swz(l16);
    auto read_h = [&](int buf, int p, int y) {
        const int cc = FP8W ? (p / PPL) * 16 + ((p % PPL) / KPH) * 8 + p % KPH : (p / PPL) * 8 + (p % PPL) * 4;
        const int ch = (cc | (FP8W ? 2 * q4 : q4)) ^ sw;
        return *(const bf16x8 *)(lds + buf * HBUF + y * 16 * HROW + l16 * HROW + ch * 16);
    };
    // half c of the 16 rows of a block from its two loads (rows 0..7, rows 8..15): lane l16 <-> row l16
    auto half_of = [&](const u32x4 &x, const u32x4 &y, int c) {
        u32x4 r;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            r[k] = c == 0 ? (uint32_t)__builtin_amdgcn_update_dpp((int)x[k], (int)y[k], 0x128 /* row_ror:8 */, 0xF, 0xC, false)
                          : (uint32_t)__builtin_amdgcn_update_dpp((int)y[k], (int)x[k], 0x128, 0xF, 0x3, false);
        return r;
    };

    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int y = 0; y < MB; ++y) acc[b][y] = f32x4{0.f, 0.f, 0.f, 0.f};

    load_h(0);
#pragma unroll
    for (int l = 0; l < LPS; ++l) load_w(0, 0, l);
    store_h(0);
    load_h(1);
#pragma unroll
    for (int l = 0; l < LPS; ++l) load_w(1, 1, l);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    bf16x8 hf[MB];
#pragma unroll
    for (int y = 0; y < MB; ++y) hf[y] = read_h(0, 0, y);

    // One slab.  The barrier before its last piece says that every wave has read the last fragments of this slab's buffer
    // and has written its part of the next slab's: so the next slab is written before it, and the one after that,
    // into this buffer, after it.  hidden_t is requested before the W_lm lines of a slab, so that the wait for it (loads
    // complete in order) leaves the W_lm loads behind it in flight.
    auto slab = [&](int it, int u) {
        store_h(u ^ 1);
        load_h(it + 2);
        __builtin_amdgcn_sched_barrier(0);
        u32x4 wh[NB];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int l = p / PPL, c = (p % PPL) / KPH, kk = p % KPH;
            if (p == NP - 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            bf16x8 wf[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (kk == 0) wh[b] = half_of(ring[u][l][b][0], ring[u][l][b][1], c);
                wf[b] = FP8W ? fp8x8_to_bf16x8(uint2{wh[b][2 * kk], wh[b][2 * kk + 1]}) : __builtin_bit_cast(bf16x8, wh[b]);
            }
#pragma unroll
            for (int y = 0; y < MB; ++y) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[b], hf[y], acc[b][y], 0, 0, 0);
                hf[y] = p + 1 < NP ? read_h(u, p + 1, y) : read_h(u ^ 1, 0, y);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (p % PPL == PPL - 1) {
                load_w(it + 2, u, l);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    int it = 0;
    for (; it + 1 < NS; it += 2) {
        slab(it, 0);
        slab(it + 1, 1);
    }
    if (it < NS) slab(it, 0);

    // ---- lane (l16, q4): verify row 16 y + l16 against vocabulary rows vw + 16 b + 4 q4 + r, ascending in (b, r)
#pragma unroll
    for (int y = 0; y < MB; ++y) {
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
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int v = vw + b * 16 + q4 * 4 + r;
                float val = acc[b][y][r];
                if (v < ve) {
                    if (a.dump && row < a.M) a.dump[(size_t)row * a.V + v] = val;
                    if (a.key) val = fmaf(val, a.inv_temp, gumbel_noise(klo, khi, (uint32_t)v));
                    if (val > bv) {      // strict >: the lowest index of the maximum
                        bv = val;
                        bi = v;
                    }
                    if (a.thr) cn += ranks_before(val, v, th, tk);
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
            red[wave][y * 16 + l16] = Best{bv, bi};
            redc[wave][y * 16 + l16] = cn;
        }
    }
    __syncthreads();
    if (tid < ROWS && m0 + tid < a.M) {
        Best best = red[0][tid];
        int32_t cn = redc[0][tid];
#pragma unroll
        for (int w = 1; w < SL_WAVES; ++w) {
            const Best o = red[w][tid];
            if (better(o.v, o.i, best.v, best.i)) best = o;
            cn += redc[w][tid];
        }
        a.part[(size_t)(m0 + tid) * a.nblocks + vt] = best;
        if (a.cnt) a.cnt[(size_t)(m0 + tid) * a.nblocks + vt] = cn;
    }
}

template <int WV, int MB, int NB, bool FP8W>
hipError_t launch_slab(const SlabTile &t, const LmHeadArgs &a, hipStream_t s)
{
    const int tm = (a.M + MB * 16 - 1) / (MB * 16);
    const dim3 grid(8u * (unsigned)tm, (unsigned)((a.nblocks + 7) / 8)), block(WV * 64);
    // W_lm that is read once, in whole lines, is not kept in L2: non-temporal
    const bool nt = tm == 1 && (FP8W ? a.d % 128 : a.d % 64) == 0;
    if (t.rot == INTERLEAVE) {          // rows of a multiple of 4096 bytes: whole lines
        if constexpr (slab_interleaves(WV, MB, FP8W)) {
            if (nt) hipLaunchKernelGGL((k_lm_head_slab<WV, MB, NB, FP8W, true, true>), grid, block, 0, s, a, t.rows, 0);
            else hipLaunchKernelGGL((k_lm_head_slab<WV, MB, NB, FP8W, false, true>), grid, block, 0, s, a, t.rows, 0);
        } else return hipErrorInvalidValue;
    } else if (nt) hipLaunchKernelGGL((k_lm_head_slab<WV, MB, NB, FP8W, true, false>), grid, block, 0, s, a, t.rows, t.rot);
    else hipLaunchKernelGGL((k_lm_head_slab<WV, MB, NB, FP8W, false, false>), grid, block, 0, s, a, t.rows, t.rot);
    return hipGetLastError();
}

template <bool FP8W>
hipError_t dispatch_slab(const SlabTile &t, const LmHeadArgs &a, hipStream_t s)
{
    switch ((t.mb * 8 + t.nb) * 32 + t.wv) {
#define AJ_SLAB(WV, MB, NB) \
    case (MB * 8 + NB) * 32 + WV: \
        if constexpr (slab_built(WV, MB, NB, FP8W)) return launch_slab<WV, MB, NB * 4 / WV, FP8W>(t, a, s); \
        break;
#define AJ_SLABS(WV, NB) \
    AJ_SLAB(WV, 1, NB) AJ_SLAB(WV, 2, NB) AJ_SLAB(WV, 3, NB) AJ_SLAB(WV, 4, NB) AJ_SLAB(WV, 5, NB) AJ_SLAB(WV, 6, NB) AJ_SLAB(WV, 7, NB) AJ_SLAB(WV, 8, NB)
        AJ_SLABS(4, 1) AJ_SLABS(4, 2) AJ_SLABS(4, 3) AJ_SLABS(4, 4) AJ_SLABS(8, 2) AJ_SLABS(8, 4) AJ_SLABS(12, 3) AJ_SLABS(16, 4)
#undef AJ_SLABS
#undef AJ_SLAB
    }
    return hipErrorInvalidValue;
}

}  // namespace aj
