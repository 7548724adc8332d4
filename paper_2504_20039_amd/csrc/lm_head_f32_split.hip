// LM head + per-block greedy maximum for fp32 storage on the bf16 matrix instructions: every fp32 operand is split exactly into
// three bf16 pieces, x = h + m + l (h and m rounded to nearest; the splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", 2019), and of the nine products of two operands six (hh, hm, mh, hl, lh, mm) are summed in
// fp32 accumulators, hh apart from the others and of each half of the row apart, so that a sum of d_t products rounds d_t / 32 times.  With x in [1, 2) |m| <= 2^-8 and |l| <= 2^-17: what
// is left out is at most 2^-24 of a product, of either sign.  (Pieces that are cut off instead leave out up to 2^-21, and always towards zero:
// 4e-8 of a sum of positive products at d_t = 2048, rounded 6e-10.)  Against 64-bit sums (2-norm), normal / positive data: 1.3e-7 / 0.9e-7 at
// d_t = 1024, 2.7e-7 / 1.7e-7 at 4096, 4.0e-7 / 2.4e-7 at 8192; the fp32 instructions of lm_head_f32.hip, which round d_t / 16 times in four partial sums,
// 2.9e-7 / 1.2e-7, 5.8e-7 / 2.4e-7, 8.1e-7 / 3.3e-7.  (In one sum per row, positive data: 1.7e-7, 3.3e-7, 4.7e-7.)
//
// What bounds it: six bf16 products take 0.4 of the time of one fp32 product on the matrix pipe, so from about 64 rows on the kernel is bound by
// the bf16 rate (816 x 2304 x 19996: 1.05 PFLOP/s of bf16 work, 667 -> 420 us), below by what a wave issues besides MFMAs: 56
// vector instructions split 8 k elements of 16 W_lm rows, next to 6 mb MFMAs (68 x 2048 x 32000: matrix pipe 36 % busy, LDS 31 %).
//   * A wave owns 16 nb vocabulary rows: whole 128-byte lines of W_lm go global -> registers, one or two slabs (of two lines) ahead,
//     take the MFMA layout by one DPP rotation per register as in lm_head_resident.hip, and are split there, a
//     block ahead of its use, between the MFMAs of the block before (sched_group_barrier: three vector instructions after each).
//   * hidden_t is split once per workgroup: the waves share the slab's fragments out, and all read the pieces from LDS, double
//     buffered, one barrier per slab.  8 waves (two per SIMD: one's vector work runs behind the other's MFMAs) share them best.
//   * Both operands are buffer loads: rows beyond V or M and k elements beyond d_t lie outside the buffer and read as zero.
//   * The matrix instructions read bf16 values below 2^-126 as zero, and values above 2^128 - 2^119 round to infinity: tiles with logits so small
//     that the one could be seen, or infinite, are computed again on the fp32 instructions (see the end of the kernel).
#include "../../include/aj.h"
#include "aj_internal.h"

namespace aj {

namespace {

constexpr int SP_LPS = 2;                       // 128-byte lines of a row (32 k elements) per slab

struct Pieces {
    bf16x8 p[3];                                // h, m, l
};

// Two fp32 values -> their upper bf16 pieces, rounded to nearest (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t round2(uint32_t a, uint32_t b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{__uint_as_float(a), __uint_as_float(b)}), b16x2));
}

// Piece K of 4 values (0: h, 1: m, rounded; 2: l, all that is left), two of them in a word; x becomes what it leaves, exactly
template <int K>
__device__ __forceinline__ uint2 piece4(u32x4 &x)
{
    if (K == 2) return uint2{__builtin_amdgcn_perm(x[1], x[0], 0x07060302), __builtin_amdgcn_perm(x[3], x[2], 0x07060302)};
    const uint2 o = {round2(x[0], x[1]), round2(x[2], x[3])};
    x = u32x4{__float_as_uint(__uint_as_float(x[0]) - __uint_as_float(o.x << 16)),
              __float_as_uint(__uint_as_float(x[1]) - __uint_as_float(o.x & 0xffff0000u)),
              __float_as_uint(__uint_as_float(x[2]) - __uint_as_float(o.y << 16)),
              __float_as_uint(__uint_as_float(x[3]) - __uint_as_float(o.y & 0xffff0000u))};
    return o;
}

template <int K>
__device__ __forceinline__ bf16x8 piece8(u32x4 &a, u32x4 &b)
{
    const uint2 p = piece4<K>(a), q = piece4<K>(b);
    return __builtin_bit_cast(bf16x8, (u32x4{p.x, p.y, q.x, q.y}));
}

// 8 fp32 values -> their three bf16 pieces
__device__ __forceinline__ Pieces split8(u32x4 a, u32x4 b)
{
    Pieces r;
    r.p[0] = piece8<0>(a, b);
    r.p[1] = piece8<1>(a, b);
    r.p[2] = piece8<2>(a, b);
    return r;
}

// D: slabs in flight (1 where two would not fit into the registers)
template <int SP_WAVES, int MB, int NB, int D, int OCC, bool NT>
__global__ __launch_bounds__(SP_WAVES * 64, OCC) void k_lm_head_f32_split(LmHeadArgs a)
{
    constexpr int ROWS = MB * 16;
    constexpr int FRAG = 1024;                                   // bytes of a fragment: 16 rows x 32 k elements
    constexpr int HBUF = SP_LPS * 3 * MB * FRAG;                 // hidden_t slab: pieces of MB row blocks x SP_LPS lines
    constexpr int UNITS = 2 * MB * SP_LPS, HU = (UNITS + SP_WAVES - 1) / SP_WAVES;   // half fragments staged per slab, per wave
    constexpr uint32_t OUT = 0x80000000u;                        // a byte offset beyond every buffer: reads as zero
    __shared__ __attribute__((aligned(1024))) char lds[2 * HBUF];
    constexpr bool HOLD = SP_WAVES == 8 || OCC == 1;             // one workgroup per compute unit: LDS for sums of half a row
    __shared__ f32x4 hold[HOLD ? NB * MB * SP_WAVES * 64 : 1];
    __shared__ Best red[SP_WAVES][ROWS];
    __shared__ int32_t redc[SP_WAVES][ROWS];
    __shared__ uint32_t redm[SP_WAVES][ROWS];                    // largest |logit|, as bits
    __shared__ uint32_t rowmax[ROWS];                            // largest |hidden_t| of a row, as bits
    __shared__ uint32_t wbits[SP_WAVES];                         // whether a wave's part of W_lm holds anything but zeros
    __shared__ int32_t again[ROWS];                              // of a row's logits, to be computed again: 1 those not finite, 2 all

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    // the row tiles of a vocabulary tile go to consecutive workgroups of one XCD (id mod 8; gridDim.x is a multiple of 8)
    const int vt = blockIdx.y * 8 + (blockIdx.x & 7), mt = blockIdx.x >> 3;
    if (vt >= a.nblocks) return;
    const int vw = (vt * SP_WAVES + wave) * 16 * NB, m0 = mt * ROWS;     // first vocabulary row of the wave
    const uint32_t rowb = (uint32_t)a.d * 4u;
    auto buffer_of = [](const void *base, uint32_t bytes) {      // in scalar registers
        const uint64_t p = (uint64_t)base;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
        return __builtin_amdgcn_make_buffer_rsrc((void *)((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes),
                                                 0x00020000);
    };
    const auto wres = buffer_of((const char *)a.W + (size_t)min(vw, a.V - 1) * rowb,
                                (uint32_t)min(max(a.V - vw, 0), 16 * NB) * rowb);
    const auto hres = buffer_of((const char *)a.H + (size_t)m0 * rowb, (uint32_t)min(a.M - m0, ROWS) * rowb);
    const int NS = (int)((rowb + SP_LPS * 128 - 1) / (SP_LPS * 128));    // slabs
    const bool weave = (rowb & 4095) == 0;
    auto slab_at = [&](int it) { return weave && it < NS ? interleave_4k<4096 / (SP_LPS * 128)>(it) : it; };

    // W_lm: load h of a block covers rows 8h .. 8h+7 x the whole 128-byte line
    const uint32_t wk = (uint32_t)(q4 + 4 * (l16 >> 3)) * 16u, wo = (uint32_t)(l16 & 7) * rowb;
    u32x4 ring[D][SP_LPS][NB][2];
    auto load_w = [&](int it, int set, int l) {
        const uint32_t kb = (uint32_t)(slab_at(it) * SP_LPS + l) * 128u + wk, kk = kb < rowb ? kb : OUT;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                ring[set][l][b][h] = __builtin_amdgcn_raw_buffer_load_b128(wres, (int)(wo + kk + (uint32_t)(b * 16 + h * 8) * rowb), 0,
                                                                        NT ? 2 : 0);
    };
    // hidden_t: unit u of a slab is half u % 2 of row block u / 2 % MB of line u / 2 / MB; lane (l16, q4) has row l16 and chunk q4 of
    // the half line, the k elements that it has of a W_lm row
    u32x4 hst[D][HU];
    const uint32_t ho = (uint32_t)l16 * rowb + (uint32_t)q4 * 16u;
    auto load_h1 = [&](int it, int set, int i) {
        const int u = min(wave + i * SP_WAVES, UNITS - 1);       // (some waves repeat the last one)
        const uint32_t kb = (uint32_t)(slab_at(it) * SP_LPS + u / (2 * MB)) * 128u + (uint32_t)(u & 1) * 64u;
        const uint32_t kk = kb + (uint32_t)q4 * 16u < rowb ? kb : OUT;
        hst[set][i] = __builtin_amdgcn_raw_buffer_load_b128(hres, (int)(ho + kk + (uint32_t)(u / 2 % MB * 16) * rowb), 0, 0);
    };
    auto load_h = [&](int it, int set) {
#pragma unroll
        for (int i = 0; i < HU; ++i) load_h1(it, set, i);
    };
    // a fragment is stored in lane order, so that reads touch every bank once (writes are of 8 bytes, 16 apart: their bank conflicts are 6 % of
    // the launch at 68 x 2048 x 32000)
    float hmax[HU];                     // largest |hidden_t| of the lane's part of the unit's row
#pragma unroll
    for (int i = 0; i < HU; ++i) hmax[i] = 0.f;
    auto store_h = [&](int buf, int set, int i) {
        const int u = min(wave + i * SP_WAVES, UNITS - 1);
        u32x4 x = hst[set][i];
        hmax[i] = fmaxf(fmaxf(hmax[i], fabsf(__uint_as_float(x[0]))), fabsf(__uint_as_float(x[1])));
        hmax[i] = fmaxf(fmaxf(hmax[i], fabsf(__uint_as_float(x[2]))), fabsf(__uint_as_float(x[3])));
        char *to = lds + buf * HBUF + u / 2 * 3 * FRAG + lane * 16 + (u & 1) * 8;
        *(uint2 *)to = piece4<0>(x);
        *(uint2 *)(to + FRAG) = piece4<1>(x);
        *(uint2 *)(to + 2 * FRAG) = piece4<2>(x);
    };
    auto read_h = [&](int buf, int l, int y, int k) {
        return *(const bf16x8 *)(lds + buf * HBUF + ((l * MB + y) * 3 + k) * FRAG + lane * 16);
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

    // the large products and the five small ones in accumulators of their own: a sum then rounds once per 32 k elements
    f32x4 acc[NB][MB], acs[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int y = 0; y < MB; ++y) acc[b][y] = acs[b][y] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A group: one block of a line
    constexpr int G = SP_LPS * NB;
    // every bit of the lane's W_lm values, to tell rows of zeros from tiny ones.  (As a statement of its own: left to itself the compiler
    // moves the values around for it, and the tiles of three blocks spill: 120 x 4096 x 24000 188 -> 224 us, so 191)
    uint32_t any = 0;
    auto split_w = [&](int set, int l, int b) {
        const u32x4 x = half_of(ring[set][l][b][0], ring[set][l][b][1], 0), y = half_of(ring[set][l][b][0], ring[set][l][b][1], 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) asm("v_or3_b32 %0, %0, %1, %2" : "+v"(any) : "v"(x[i]), "v"(y[i]));
        return split8(x, y);
    };

    for (int r = tid; r < ROWS; r += SP_WAVES * 64) rowmax[r] = 0;
    bf16x8 hf[MB][3];
    load_h(0, 0);
#pragma unroll
    for (int i = 0; i < D; ++i) {
        if (i + 1 < D) load_h(i + 1, i + 1);
#pragma unroll
        for (int l = 0; l < SP_LPS; ++l) load_w(i, i, l);
    }
#pragma unroll
    for (int i = 0; i < HU; ++i) store_h(0, 0, i);
    load_h(D, 0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int y = 0; y < MB; ++y)
#pragma unroll
        for (int k = 0; k < 3; ++k) hf[y][k] = read_h(0, 0, y, k);
    Pieces w = split_w(0, 0, 0);
    if (NB == 1) load_w(D, 0, 0);

    // One slab.  The next group is split behind the MFMAs of a group.  The barrier before the last group says that every wave
    // has read the last fragments of this slab's buffer and has written its part of the next slab's: the next slab is
    // written before it, and the one after that, into this buffer, after it.
    auto slab = [&](int it, int u) {
        const int un = (u + 1) % D, buf = it & 1;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int l = g / NB, b = g % NB;
            if (g == G - 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const int gn = (g + 1) % G, ln = gn / NB;
            const Pieces wn = split_w(g + 1 < G ? u : un, ln, gn % NB);
#pragma unroll
            for (int i = 0; i < HU; ++i)
                if (g == i % (G - 1)) {
                    store_h(buf ^ 1, un, i);
                    load_h1(it + 1 + D, un, i);
                }
            if (gn % NB == NB - 1) load_w(g + 1 < G ? it + D : it + 1 + D, g + 1 < G ? u : un, ln);   // the line's registers are free
            // small products first; a fragment's last use in the line is followed by the read of the next line's
#pragma unroll
            for (int kh = 2; kh >= 0; --kh)
#pragma unroll
                for (int kw = 2 - kh; kw >= 0; --kw)
#pragma unroll
                    for (int y = 0; y < MB; ++y) {
                        f32x4 &c = kh + kw == 0 ? acc[b][y] : acs[b][y];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.p[kw], hf[y][kh], c, 0, 0, 0);
                        if (kw == 0 && b == NB - 1)
                            hf[y][kh] = l + 1 < SP_LPS ? read_h(buf, l + 1, y, kh) : read_h(buf ^ 1, 0, y, kh);
                    }
#pragma unroll
            for (int i = 0; i < 6 * MB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // an MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);      // vector instructions
            }
            __builtin_amdgcn_sched_barrier(0);
            w = wn;
        }
    };
    // The large products of the first and the second half of the row are sums of their own: partial sums, and what they round by, stay half as
    // large.  The first half's are put aside in LDS where there is room for them (in registers the largest tiles have none: 480 x
    // 1024 x 50257 326 -> 367 us, in LDS 327)
    f32x4 half[NB][MB];
    auto held = [&](int b, int y) -> f32x4 & { return HOLD ? hold[(b * MB + y) * (SP_WAVES * 64) + tid] : half[b][y]; };
    int it = 0;
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {
        const int end = part ? NS : NS / 2;
#pragma unroll 1
        for (; it + D <= end; it += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) slab(it + i, i);
        }
        if (part == 0) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int y = 0; y < MB; ++y) {
                    held(b, y) = acc[b][y];
                    acc[b][y] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    }
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (it + i < NS) slab(it + i, i);

#pragma unroll
    for (int i = 0; i < HU; ++i) {
        const float m = fmaxf(hmax[i], __shfl_xor(hmax[i], 16));
        const float n = fmaxf(m, __shfl_xor(m, 32));
        if (q4 == 0) atomicMax(&rowmax[min(wave + i * SP_WAVES, UNITS - 1) / 2 % MB * 16 + l16], __float_as_uint(n));
    }
    const bool live = __any((any << 1) != 0);      // (without the signs)
    if (lane == 0) wbits[wave] = live;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int y = 0; y < MB; ++y) acc[b][y] = (acc[b][y] + acs[b][y]) + held(b, y);

    // ---- lane (l16, q4): verify row 16 y + l16 against vocabulary rows vw + 16 b + 4 q4 + r, ascending in (b, r)
    for (bool second = false;; second = true) {
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
            uint32_t bm = 0;             // largest |logit|, as bits: NaN above infinity above all others
            int32_t bi = 0x7fffffff, cn = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int v = vw + b * 16 + q4 * 4 + r;
                    float val = acc[b][y][r];
                    bm = max(bm, __float_as_uint(fabsf(val)));
                    if (v < a.V) {
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
                bm = max(bm, (uint32_t)__shfl_xor((int)bm, off));
            }
            if (q4 == 0) {
                red[wave][y * 16 + l16] = Best{bv, bi};
                redc[wave][y * 16 + l16] = cn;
                redm[wave][y * 16 + l16] = bm;
            }
        }
        __syncthreads();
        int redo = 0;
        if (tid < ROWS && m0 + tid < a.M) {
            Best best = red[0][tid];
            int32_t cn = redc[0][tid];
            uint32_t bm = redm[0][tid], live = wbits[0];
#pragma unroll
            for (int w = 1; w < SP_WAVES; ++w) {
                const Best o = red[w][tid];
                if (better(o.v, o.i, best.v, best.i)) best = o;
                cn += redc[w][tid];
                bm = max(bm, redm[w][tid]);
                live |= wbits[w];
            }
            a.part[(size_t)(m0 + tid) * a.nblocks + vt] = best;
            if (a.cnt) a.cnt[(size_t)(m0 + tid) * a.nblocks + vt] = cn;
            // The matrix instructions take bf16 values below 2^-126 as zero.  What that may leave out of a logit is less than
            // d 2^-126 (1 + the row's largest |hidden_t|), and 2^-36 of the product of the norms unless the row itself is tiny: next
            // to a tile whose largest |logit| reaches 2^-85 (1 + ...), nothing.  Below it the tile is computed again,
            // unless all of its W_lm rows are zero, as the padding of a vocabulary is (68 x 2048 x 32000 with 512 such rows: 280 us with the
            // second pass, 78 without).
            // A piece that rounds to infinity (values above 2^128 - 2^119) makes all of its logits infinite or NaN, and so do products
            // that overflow: those logits are computed again too, alone of their row.
            const float hm = __uint_as_float(rowmax[tid]);
            if (!second) {
                if (bm >= 0x7f800000u) redo = 1;
                else if (live && hm > 0.f && (hm < 0x1p-90f || __uint_as_float(bm) < 0x1p-85f * fmaxf(hm, 1.f))) redo = 2;
            }
            again[tid] = redo;
        }
        if (second || !__syncthreads_or(redo)) break;

        // the rows in question once more on the fp32 matrix instructions, which keep such values: never reached by logits of a
        // normal size, so neither pipelined nor shared through LDS
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int y = 0; y < MB; ++y) acs[b][y] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (uint32_t k0 = 0; k0 < rowb; k0 += 64) {
            const uint32_t k = k0 + (uint32_t)q4 * 16u, kk = k < rowb ? k : OUT;
            f32x4 h[MB];
#pragma unroll
            for (int y = 0; y < MB; ++y)
                h[y] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(hres, (int)((uint32_t)(y * 16 + l16) * rowb + kk), 0, 0));
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, (int)((uint32_t)(b * 16 + l16) * rowb + kk), 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int y = 0; y < MB; ++y) acs[b][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], h[y][e], acs[b][y], 0, 0, 0);
            }
        }
#pragma unroll
        for (int y = 0; y < MB; ++y) {
            const int which = m0 + y * 16 + l16 < a.M ? again[y * 16 + l16] : 0;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool finite = (__float_as_uint(acc[b][y][r]) & 0x7fffffffu) < 0x7f800000u;
                    acc[b][y][r] = which == 2 || (which == 1 && !finite) ? acs[b][y][r] : acc[b][y][r];
                }
        }
    }
}

// ---- launch
template <int WV, int MB, int NB, int D, int OCC>
hipError_t launch(const LmHeadArgs &a, hipStream_t s)
{
    const int tm = (a.M + MB * 16 - 1) / (MB * 16);
    const dim3 grid(8u * (unsigned)tm, (unsigned)((a.nblocks + 7) / 8));
    // W_lm that is read once, in whole lines, is not kept in L2: non-temporal
    if (tm == 1 && a.d % 32 == 0) hipLaunchKernelGGL((k_lm_head_f32_split<WV, MB, NB, D, OCC, true>), grid, dim3(WV * 64), 0, s, a);
    else hipLaunchKernelGGL((k_lm_head_f32_split<WV, MB, NB, D, OCC, false>), grid, dim3(WV * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace

// The tile that costs least, and whether it beats the fp32 kernel (old_cost, us).  Measured on 685 problems (d_t 256 .. 8192, V
// 4096 .. 152064, 9 .. 1000 rows): launch 3 us + rounds of tiles over the compute units x (5 us + (c0 + c1 mb) d_t / 1000), to 8 %.
// The fp32 kernel keeps what is bound by the W_lm stream or by the latency of a short problem: up to 32 rows (17 x 2048 x 107552: 166 us,
// here 166; 9 x 1024 x 32000: 21, 27), vocabularies that are too few tiles (33 x 4096 x 16000: 64, 81), and what the model puts within
// 14 % (20 % with 3 row blocks): between, either may win.  Beyond, the median is 0.69 of a whole call's time: 68 x 2048 x 32000 94 -> 69
// (kernel alone), 272 x 4096 x 32000 650 -> 394, 1000 x 2048 x 16000 549 -> 353, 68 x 256 x 128256 84 -> 48.  Below 256 elements not measured
// (4 slabs: filling and emptying the pipeline would be half of the loop).
bool lm_head_f32_split_plan(int M, int V, int d, int num_cus, double old_cost, F32SplitTile *tile)
{
    static const struct { int wv, nb, mb0, mb1; double c0, c1; } T[5] = {       // (the row blocks for which a tile can be cheapest)
        {4, 1, 3, 5, 5.4, 2.5}, {4, 2, 3, 4, 8.3, 4.3}, {4, 3, 3, 5, 14.0, 5.1}, {8, 1, 5, 5, 15.3, 2.7}, {8, 2, 3, 5, 25.8, 3.5}};
    const int blocks = (M + 15) / 16, cus = (num_cus + 7) / 8;
    if (blocks < 3 || d < 256 || d > 1 << 20) return false;
    double best = 0.0;
    for (const auto &t : T)
        for (int mb = blocks < 5 && blocks > t.mb0 ? blocks : t.mb0; mb <= t.mb1 && mb <= blocks; ++mb) {
            const int rows = 16 * t.wv * t.nb, nblocks = (V + rows - 1) / rows, tm = (blocks + mb - 1) / mb;
            // the row tiles of a vocabulary tile go to one of the 8 XCDs: its share of tiles over its share of compute units
            const int64_t rounds = ((int64_t)(nblocks + 7) / 8 * tm + cus - 1) / cus;
            const double cost = 2.9 + (double)rounds * (5.1 + (t.c0 + t.c1 * mb) * d / 1000.0);
            if (best == 0.0 || cost < best) {
                best = cost;
                *tile = F32SplitTile{t.wv, t.nb, mb};
            }
        }
    return best < (blocks == 3 ? 0.80 : 0.86) * old_cost;
}

hipError_t lm_head_f32_split(const F32SplitTile &t, const LmHeadArgs &a, hipStream_t s)
{
    if (a.M <= 0) return hipSuccess;
    switch (t.wv * 64 + t.nb * 8 + t.mb) {
#define AJ_SPLIT(WV, NB, MB, D, OCC) case WV * 64 + NB * 8 + MB: return launch<WV, MB, NB, D, OCC>(a, s);
        AJ_SPLIT(4, 1, 3, 2, 2) AJ_SPLIT(4, 1, 4, 2, 2) AJ_SPLIT(4, 1, 5, 1, 2)
        AJ_SPLIT(4, 2, 3, 2, 1) AJ_SPLIT(4, 2, 4, 2, 1)
        AJ_SPLIT(4, 3, 3, 2, 1) AJ_SPLIT(4, 3, 4, 2, 1) AJ_SPLIT(4, 3, 5, 2, 1)
        AJ_SPLIT(8, 1, 5, 2, 2)
        AJ_SPLIT(8, 2, 3, 1, 2) AJ_SPLIT(8, 2, 4, 1, 2) AJ_SPLIT(8, 2, 5, 1, 2)
#undef AJ_SPLIT
        default: return hipErrorInvalidValue;
    }
}

}  // namespace aj
