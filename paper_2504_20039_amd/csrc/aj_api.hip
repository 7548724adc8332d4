// C ABI of libaj (declared in include/aj.h): argument checks, workspace, kernel dispatch.
#include <math.h>
#include <mutex>
#include <new>

#include "../../include/aj.h"
#include "aj_internal.h"

using namespace aj;

constexpr int VARIANT_SLAB = -2, VARIANT_F32_SPLIT = -3;

struct aj_handle {
    aj_config cfg;
    int M;
    int variant;   // AJ_KERNEL_* actually used (for bf16), -1 for the fp32 kernel, VARIANT_F32_SPLIT for the one on bf16 instructions,
                   // VARIANT_SLAB for the small-tile kernel
    bool stream16; // AJ_KERNEL_STREAM served by the 16-row-tile kernel
    bool fp8w;     // W_lm stored as FP8 E4M3 (16-row-tile, accumulator-resident, wide and small-tile kernels)
    SlabTile slab; // tile of the small-tile kernel
    F32SplitTile split;
    int row_blocks; // AJ_KERNEL_PAIR9: verify rows per tile / 32
    int nblocks;   // partials per verify row
    int device;
    int num_cus;
    Best *part;    // [M][nblocks]
    int32_t *t_star;
    float *maxlogit;
    float *score;  // [2][B][K] or nullptr
    uint8_t *rej;  // [B][K] rejected-slot flags (tail kernels' split form)
    float *zt;     // [M] fused judge row's logits (AJ_FLAG_FUSED_JUDGE)
    // top-K baseline workspace (AJ_FLAG_TOPK)
    int32_t *cnt;      // [M][nblocks]
    float *thr;        // [M]
    int32_t *thr_tok;  // [M]
    int32_t *rank;     // [M]
    hipEvent_t ev[64][2];
    bool ev_ok;
    uint64_t calls;
};

static thread_local int g_last_hip = 0;

static int hip_fail(hipError_t e)
{
    g_last_hip = (int)e;
    return AJ_EHIP;
}

extern "C" int aj_last_hip_error(void) { return g_last_hip; }

extern "C" const char *aj_strerror(int status)
{
    switch (status) {
        case AJ_OK: return "ok";
        case AJ_EINVAL: return "invalid argument (null/misaligned pointer, bad shape, or tau outside [0,1])";
        case AJ_ENOMEM: return "device workspace allocation failed";
        case AJ_EHIP: return "a HIP call failed (see aj_last_hip_error)";
        case AJ_ESTATE: return "call not valid for this handle";
        case AJ_ELIMIT: return "the shape needs more workspace than the static buffer of aj_verify_static holds";
        default: return "unknown status";
    }
}

static bool aligned16(const void *p) { return (((uintptr_t)p) & 15u) == 0; }

static void free_all(aj_handle *h)
{
    if (h->part) (void)hipFree(h->part);
    if (h->t_star) (void)hipFree(h->t_star);
    if (h->maxlogit) (void)hipFree(h->maxlogit);
    if (h->score) (void)hipFree(h->score);
    if (h->rej) (void)hipFree(h->rej);
    if (h->zt) (void)hipFree(h->zt);
    if (h->cnt) (void)hipFree(h->cnt);
    if (h->thr) (void)hipFree(h->thr);
    if (h->thr_tok) (void)hipFree(h->thr_tok);
    if (h->rank) (void)hipFree(h->rank);
    if (h->ev_ok)
        for (int i = 0; i < 64; ++i) {
            (void)hipEventDestroy(h->ev[i][0]);
            (void)hipEventDestroy(h->ev[i][1]);
        }
}

// The small-tile kernel (lm_head_slab.h): the tile for which the busiest compute unit has least to do, and what that costs in
// rounds of tiles over the compute units times the cost of a round.  Costs of a round are microseconds at d_t = 7168 (less
// 9 us of launches and tail); from d_t = 1024 on they grow with d_t about alike in all kernels, so that their ratios
// decide (below, see slab_wins).  Measured on V = 17000 .. 128256
// (bf16 / FP8): 64 nb vocabulary rows x 16 mb verify rows take 25 + 4.5 mb / 14 + 4 mb with nb = 1, 58 + 4.5 mb / 28 + 6 mb
// with nb = 2, 92 + 4 mb / 44 + 7.5 mb with nb = 3, 105 + 5 mb / 50 + 14 mb with nb = 4.  (99 rows x 7168 x 36000, nb = 4, 3, 2: 240
// / 132 / 175 us; 48 rows x 17000: 126 / 105 / 77; 60 rows x 2888 x 50257: 86 / 120 / 89; 264 rows x 16000, nb = 3: 252 tiles in three
// row tiles, 33 of them on an XCD of 32 compute units, 189 us; nb = 4: 24 at most, 149.)
struct SlabPlan {
    SlabTile tile;
    int nblocks, rounds;
    double cost;
};
static SlabPlan slab_plan(int M, int V, int d, bool fp8w, int num_cus)
{
    static const struct { int nb, max_mb; double bf16[2], fp8[2]; } T[4] = {
        {4, 6, {105, 5.0}, {50, 14.0}}, {3, 8, {92, 4.0}, {44, 7.5}}, {2, 8, {58, 4.5}, {28, 6.0}}, {1, 4, {25, 4.5}, {14, 4.0}}};
    const int blocks = (M + 15) / 16;
    SlabPlan best = {};
    for (const auto &t : T) {
        const int tm = (blocks + t.max_mb - 1) / t.max_mb, mb = (blocks + tm - 1) / tm;
        if (t.nb == 1 && tm > 1) continue;      // 64 x 64 tiles: twice the time of 128 x 128 per logit
        const int nblocks = (V + 64 * t.nb - 1) / (64 * t.nb);
        // the row tiles of a vocabulary tile go to one of the 8 XCDs: its share of tiles over its share of compute units
        const int cus = (num_cus + 7) / 8, rounds = (int)(((int64_t)(nblocks + 7) / 8 * tm + cus - 1) / cus);
        const double *c = fp8w ? t.fp8 : t.bf16, cost = rounds * (c[0] + c[1] * mb);
        if (best.nblocks && cost >= best.cost) continue;
        // One round: many waves of one block each (lm_head_slab.h; FP8 with up to two row blocks, or tiles of 256 rows, 4 as before:
        // 33 x 4096 x 50257 1.04; and tiles of 128 x 96 rows: 96 x 4096 x 32312 50.5 us, 4 waves 46.7; 178 x 7168 x 16192 76, 72).  More: 4 waves, two
        // workgroups per compute unit
        const bool many = rounds == 1 && t.nb > 1 && (!fp8w || (mb > 2 && t.nb < 4 && !(t.nb == 2 && mb == 6)));
        // Full tiles of 256 rows, a power of two bytes apart, with little work per byte: 4 waves too (45 x 2048 x 65130 50.6, 16 waves 53.5; 38 x 4096 x
        // 62914 84, 87; 8 x 8192 x 65536 160, 164; but 62 x 8192 x 65536 0.97 with 16, lower tiles and other row lengths 0.93)
        const bool full = !fp8w && t.nb == 4 && mb <= 5 && mb * d <= 12288 && d >= 2048 && (d & (d - 1)) == 0 && V > 60 * 4 * num_cus;
        const int wv = !many || full ? 4 : t.nb == 4 && mb > 4 ? 8 : 4 * t.nb;
        if (!slab_built(wv, mb, t.nb, fp8w)) continue;       // (never where it would be the cheapest, with 256 compute units)
        // The tiles of these rounds that share the vocabulary out evenly.  Not where there are many (their last, partial round is a small
        // part, and tiles bound by the matrix pipe would only compute more rows for nothing: 2000 x 2888 x 100000 1.05)
        const int most = 8 * (rounds * cus / tm), cap = 64 * t.nb / wv;
        const int even = (V + wv * most - 1) / (wv * most), rows = rounds <= (tm == 1 ? 8 : 2) && even < cap ? even : cap;
        best = {{mb, t.nb, 0, wv, rows}, (V + wv * rows - 1) / (wv * rows), rounds, cost};
    }
    return best;
}

// Whether AJ_KERNEL_AUTO takes the small-tile kernel instead of h->variant, the choice among the others (measured on both
// sides, us, other kernel -> small tiles).
//   * Hidden sizes that are not a multiple of 32: up to 64 rows always, beyond from d_t = 320 on (the general kernel: 60 rows x 2888 x
//     50257 123 -> 86, 2000 rows 999 -> 758).  In shorter rows the reduction of a tile, two workgroups at a time, outweighs
//     its loop: 2000 rows x 72 x 100000 142 -> 208, 128 rows x 264 x 50257 23.0 -> 24.9; 128 x 328 x 65536 equal.
//   * Other hidden sizes that are not a multiple of 128: the same up to 128 rows (36 rows x 4160: V = 17000 100 -> 46, V = 128256
//     237 -> 178), but 113 .. 128 rows only when their rounds cost less than those of 256 x 256 tiles, 185 (128 rows x 4160:
//     V = 72000 0.73 of the time, V = 128256 244 -> 257; 352 x 128256 1.06 of it); up to 256 rows when one round of tiles does it
//     (200 rows x 4160, V = 17000 106 -> 80; V = 50257, three rounds: 124 -> 186).  Multiples of 128 only: the streaming tiles
//     keep up to 128 rows.
//   * Multiples of 256 up to 272 rows: when its rounds cost less than those of the accumulator-resident kernel (512 vocabulary
//     rows per compute unit and pass: 192 + 5 mb + V / 7000 as more of them share the HBM, FP8 98 + 4 mb and 15 more from 6 row
//     blocks on) or of the wide kernel (256
//     per tile: 107 + 4.2 mb, FP8 27 + 7.6 mb).  A vocabulary of 17000 is 34 or 67 workgroups there, for 256 compute
//     units: 24 rows x 7168 208 -> 67, 264 rows 182 -> 153; 122 rows x 72000 (282 wide tiles, a second
//     round of 26) 302 -> 251; at V = 128256 they all have work: 272 -> 282.
//     Many rounds of the smallest tiles run into the rate at which they stream W_lm, V / 465 (V / 400 with rows a power of two
//     apart).  Below d_t = 1024, what a round costs whatever its row length (the reduction) is added on both sides: 100 rows x
//     256 x 152064 35.8 -> 46.0, 64 rows x 256 x 65536 19.7 -> 20.6, 100 x 256 x 32000 21.7 -> 19.9, 48 x 512 x 50257 26.4 -> 22.8.
//     The costs are those of tiles of full height; the even ones (slab_plan) take less of it: the factors, below which no shape of 1167
//     (3 .. 264 rows, d_t 1024 .. 7168, V 16000 .. 152064) loses more than 2 % against the other kernel, median 0.92 (48 x 4096 x 90000 0.89,
//     144 x 4096 x 72000 0.89; FP8 33 x 4096 x 152064 0.75, 264 x 4096 x 24000 0.83).  In rows of a power of two at 65..112 rows the k order of
//     the tiles can meet on the memory channels (99 x 4096 x 80000: 163 us, 42 instead of 40 rows per wave 133): not taken there.
//     W_lm bound: 2 rows x 7168, V = 96000 224 -> 205; d_t = 3072, V = 100000 102 -> 106; d_t = 8192, V = 100000 248 -> 294.
static bool slab_wins(const aj_handle *h, const SlabPlan &p)
{
    const int M = h->M, V = h->cfg.V, d = h->cfg.d_t, mb = (M + 15) / 16;
    // V < 12288 is not where the small tiles stop paying, only where they have been taken so far (the smallest vocabularies of
    // the models in use have 16000): below it they are faster as well (64 rows x 4096 x 8000: accumulator-resident kernel 128 us, small
    // tiles 36; 17 x 2888 x 8000: general kernel 73, 20; 264 x 4096 x 12000: wide kernel 110, 72), except at a vocabulary of one
    // tile (100 rows x 512 x 64: 17.6, 19.8).  The tests of the other kernels reach them through AJ_KERNEL_AUTO there and would
    // have to force them first.  d_t: 32-bit offsets within a tile
    if (V < 12288 || d > 1 << 20 || !p.nblocks) return false;
    // never more workspace than the static entry point has, unless the other kernel needs as much
    if ((uint64_t)M * p.nblocks * sizeof(Best) + 12ull * M + 1024 > AJ_STATIC_SCRATCH_BYTES && p.nblocks > h->nblocks) return false;
    const double fixed = d < 1024 ? 7168.0 / d - 7.0 : 0.0;
    const bool long_rows = M <= 64 || d >= 320, pow2 = (d & (d - 1)) == 0;
    switch (h->variant) {
        case AJ_KERNEL_TILE: return long_rows;
        case AJ_KERNEL_BIG:
        case AJ_KERNEL_TALL:
            if (!long_rows) return false;
            if (d % 128 != 0 && M <= 128) return mb < 8 || p.cost < 185.0 * ((h->nblocks + h->num_cus - 1) / h->num_cus);
            return M <= 256 && p.rounds == 1;
        case AJ_KERNEL_RESIDENT: {
            const int64_t pass = (int64_t)h->nblocks * 512;
            const double c = h->fp8w ? 98 + 4.0 * mb + (mb > 5 ? 15 : 0) + (mb > 7 ? 25 : 0) : 192 + 5.0 * mb + V / 7000.0;
            // (FP8: many rounds of the smallest tiles at nearly full height gain little from it: 30 x 2048 x 78643 45.8 us, other kernel 42.8; 30 x
            // 3072 x 73728 61.1, 59.7; 30 x 7168 x 78643 is the exception, 0.95)
            const bool low = p.tile.nb > 1 || p.tile.wv * p.tile.rows < 60;
            const double even = d < 2048 ? 1.0 : h->fp8w ? (low ? 0.86 : 0.97) : mb < 5 || !pow2 ? 0.9 : 1.0;
            const double stream = h->fp8w ? 0.0 : V / (pow2 ? 400.0 : 465.0);
            const double tiles = even * p.cost + p.rounds * (0.5 * p.tile.mb * p.tile.nb + 0.3) * fixed;
            return (tiles > stream ? tiles : stream) < (c + 0.5 * mb * fixed) * (double)((V + pass - 1) / pass);
        }
        case AJ_KERNEL_WIDE:
            // (Rows of a power of two: the interleaved k order gives the wide kernel most, 0.78 .. 0.96 of the time behind its cost: 126 x 8192 x
            // 152064 512 us, small tiles 544; 144 x 8192 x 72000 334, 340; 4096 175, 175.  Other multiples of 2048, interleaved too, are like the rest:
            // 144 x 6144 x 72000 301 us, small tiles 276; 10240 499, 459; 12288 594, 536; 7168 312, 303; 16384 like 8192: 150 x 72000 654, 664)
            return (h->fp8w ? 0.8 : !pow2 || d < 2048 ? 0.84 : d < 8192 ? 0.97 : 1.0) * p.cost <
                   (h->fp8w ? 27 + 7.6 * mb : 107 + 4.2 * mb) * (double)((h->nblocks + h->num_cus - 1) / h->num_cus);
        default: return false;
    }
}


// Whether AJ_KERNEL_AUTO takes two row tiles of 160 verify rows instead of the wide kernel's one (161 .. 272 rows): where the vocabulary is so
// few tiles of 256 that a round of one row tile leaves half of the compute units without work, and the small tiles do not fill them better.
// Costs as in slab_wins, this one's 142 (whole calls, us, wide kernel or small tiles -> this: 264 rows x 4096 x 24000 113 -> 79, 264 x 7168 x 32000
// 199 -> 146, 200 x 4096 x 32000 102 -> 83, 165 x 7168 x 32000 140 -> 135, 264 x 7168 x 21700 187 -> 137, 264 x 1024 x 21700 45 -> 31; 240 x 24000 stays with the
// small tiles, 122 against 135, and 264 x 7168 x 18000, 126 against 134).  Rows under 1024 elements not measured.
static bool two_row_tiles_win(const aj_handle *h, const SlabPlan &p)
{
    const aj_config &c = h->cfg;
    if (h->variant != AJ_KERNEL_WIDE || h->fp8w || h->M <= 160 || c.V < 12288 || c.d_t < 1024) return false;
    const int tiles = 2 * ((c.V + 255) / 256);
    if (tiles > h->num_cus || !lm_head_pair9_supports(h->M, c.V, c.d_t)) return false;
    return 142.0 < 0.84 * p.cost && 142.0 < 107 + 4.2 * ((h->M + 15) / 16);
}

// Validate a configuration and choose the LM-head kernel for it on the current device: fills everything of *h
// that is not a device allocation.  Allocates nothing.
static int plan_handle(const aj_config &c, aj_handle *h)
{
    if (c.dtype != AJ_F32 && c.dtype != AJ_BF16) return AJ_EINVAL;
    const int mult = c.dtype == AJ_BF16 ? 8 : 4;
    if (c.B < 0 || c.K < 1 || c.K > 1023 || c.V < 1 || c.d_t < mult || c.d_d < 0) return AJ_EINVAL;
    if (c.d_t % mult || c.d_d % mult) return AJ_EINVAL;
    if (c.feat_offset != 0 && c.feat_offset != 1) return AJ_EINVAL;
    if (c.kernel < AJ_KERNEL_AUTO || c.kernel > AJ_KERNEL_WIDE) return AJ_EINVAL;
    if ((int64_t)c.B * (c.K + 1) > (int64_t)1 << 24) return AJ_EINVAL;
    // vocabulary indices go through 24-bit multiplies (tile offsets, the sampling generator's first step)
    if (c.V >= (1 << 24)) return AJ_EINVAL;

    if (c.flags & ~(AJ_FLAG_DEBUG | AJ_FLAG_PROFILE | AJ_FLAG_TOPK | AJ_FLAG_FUSED_JUDGE)) return AJ_EINVAL;
    h->cfg = c;
    h->M = c.B * (c.K + 1);
    hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) return hip_fail(e);
    e = hipDeviceGetAttribute(&h->num_cus, hipDeviceAttributeMultiprocessorCount, h->device);
    if (e != hipSuccess) return hip_fail(e);
    if (c.w_dtype != AJ_W_SAME && c.w_dtype != AJ_W_FP8_E4M3) {
        return AJ_EINVAL;
    }
    if (c.w_dtype == AJ_W_FP8_E4M3) {
        // FP8 weights: the kernels that stream W_lm straight into registers (up to 272 verify rows; beyond that the path
        // is bound by the matrix pipe and the bytes of W_lm cost no time), and no top-K baseline (its pre-pass reads
        // W_lm rows)
        if (c.dtype != AJ_BF16 || (c.flags & (AJ_FLAG_TOPK | AJ_FLAG_FUSED_JUDGE))) return AJ_EINVAL;
        const bool s16 = (c.kernel == AJ_KERNEL_AUTO || c.kernel == AJ_KERNEL_STREAM) &&
                         lm_head_stream16_fp8w_supports(h->M, c.V, c.d_t);
        const bool res = (c.kernel == AJ_KERNEL_AUTO || c.kernel == AJ_KERNEL_RESIDENT) &&
                         lm_head_resident_supports(h->M, c.V, c.d_t, true);
        const bool wide = (c.kernel == AJ_KERNEL_AUTO || c.kernel == AJ_KERNEL_WIDE) &&
                          lm_head_wide_supports(h->M, c.V, c.d_t, true);
        if (h->M > 0 && !s16 && !res && !wide) return AJ_EINVAL;
        h->fp8w = true;
        if (s16 || h->M == 0) {
            h->variant = AJ_KERNEL_STREAM;
            h->stream16 = true;
            h->nblocks = lm_head_stream16_blocks(c.V, h->num_cus);
        } else if (res && !(wide && h->M > 112 && c.kernel == AJ_KERNEL_AUTO)) {     // (113..128 rows: see the bf16 rule below)
            h->variant = AJ_KERNEL_RESIDENT;
            h->nblocks = lm_head_resident_blocks(c.V, h->num_cus);
        } else {
            h->variant = AJ_KERNEL_WIDE;
            h->nblocks = lm_head_wide_blocks(c.V);
        }
    } else if (c.dtype == AJ_F32) {
        if (c.kernel != AJ_KERNEL_AUTO || (c.flags & AJ_FLAG_FUSED_JUDGE)) {
            return AJ_EINVAL;
        }
        if (c.V > 65535 * 64) return AJ_EINVAL;
        h->variant = -1;
        h->nblocks = lm_head_f32_blocks(h->M, c.V, c.d_t, h->num_cus);
        if (h->M > 0 && lm_head_f32_split_plan(h->M, c.V, c.d_t, h->num_cus, lm_head_f32_cost(h->M, c.V, c.d_t, h->num_cus), &h->split)) {
            const int rows = 16 * h->split.wv * h->split.nb;
            h->variant = VARIANT_F32_SPLIT;
            h->nblocks = (c.V + rows - 1) / rows;       // never more than the fp32 kernel's, whose tiles have 64 rows at most
        }
    } else {
        int v = c.kernel;
        h->row_blocks = 9;
        if (v == AJ_KERNEL_AUTO) {
            // W_lm-streaming kernels up to 128 verify rows: the 16-row-tile kernel with hidden_t in registers
            // (<= 32 rows, d_t = 2048 or 4096), else the kernel that keeps the logits in registers (d_t % 256 == 0, <= 112 rows), else
            // 128-vocabulary tiles of 32, 64 or 128 rows with a running maximum.  113..272 rows: the wide kernel.
            // Above that, the large-tile kernel that has the busiest compute unit do least: rounds of tiles x rows of a tile (padded rows are
            // wasted MFMA work, an empty last round wasted time) x a per-row factor against the 256-row whole-line kernel (PAIR =
            // 1).  Measured at d_t = 1024, 4096, 8192, V = 32000 and 128256, 288 .. 8320 rows: tiles of 288 rows 1.17, 1.04, 1.03 (an epilogue that spills), 224 1.03 .. 1.08,
            // 192 1.06 .. 1.11, 160 1.15 .. 1.3 (two row tiles each stream W_lm), the 256-row kernel with 64-byte pieces 1.09 .. 1.11, the 8-wave 288/320-row
            // kernel 1.19 .. 1.26.  Whole calls, us, PAIR -> chosen: 396 rows x 4096 x 128256 415 -> 392 (224), 380 rows 412 -> 358 (192), 672 x 4096 x
            // 32000 210 -> 170 (192), 600 207 -> 154 (160), 300 (8-wave kernel) 144 -> 89 (160), 1056 x 4096 x 128256 (288 rows) 949 -> 915 (224).
            // A batch of 257..320 rows in ONE row tile reads W_lm from HBM only once.  Vocabularies under 12288 go by the padded rows alone, as
            // before (the tests of the other kernels reach them there), and so do hidden sizes that are no multiple of 256.
            // The general kernel is left with hidden sizes that are not a multiple of 32 and with up to
            // 128 rows at multiples of 32 only.  Where small tiles do better, slab_wins() below takes the call from the kernel
            // chosen here.
            if (lm_head_stream16_supports(h->M, c.V, c.d_t)) {
                v = AJ_KERNEL_STREAM;
            } else if (h->M <= 112 && lm_head_resident_supports(h->M, c.V, c.d_t, false)) {
                v = AJ_KERNEL_RESIDENT;     // up to 112 rows at any hidden size that is a multiple of 256
            } else if (lm_head_wide_supports(h->M, c.V, c.d_t, false)) {
                // 113..272 rows: W_lm straight into registers, 16-row blocks, one row tile (0.37 ms against 0.46 of a padded
                // 256-row tile at 144 rows of the 70B shape, 0.51 against 0.55 of the 288-row tile at 264; at 8 row blocks 0.36
                // against the 0.40 of the accumulator-resident kernel, which is short of registers there)
                v = AJ_KERNEL_WIDE;
            } else if (lm_head_resident_supports(h->M, c.V, c.d_t, false)) {
                v = AJ_KERNEL_RESIDENT;     // 113..128 rows where the wide kernel does not apply (a vocabulary under 256)
            } else if (lm_head_mfma_supports(AJ_KERNEL_STREAM, h->M, c.V, c.d_t)) {
                v = AJ_KERNEL_STREAM;
            } else {
                const bool pair = lm_head_pair_supports(h->M, c.V, c.d_t);
                const bool rounds = pair && c.V >= 12288;
                // rows of matrix work per compute unit (see above) or, without rounds, in all
                auto work = [&](int padded, int tile_rows) {
                    const int64_t tiles = (int64_t)(padded / tile_rows) * ((c.V + 255) / 256);
                    const double whole = (double)((tiles + h->num_cus - 1) / h->num_cus), part = (double)tiles / h->num_cus;
                    // (of many rounds the last, partial one costs about half of its empty share)
                    return rounds ? (whole > 8 ? (whole + part) / 2 : whole) * tile_rows : (double)padded;
                };
                const int tall = lm_head_mfma_padded_rows(AJ_KERNEL_TALL, h->M), tall_rows = tall < (h->M + 319) / 320 * 320 ? 288 : 320;
                struct { int kernel, row_blocks; bool ok; double cost; } cand[7] = {
                    {AJ_KERNEL_PAIR, 0, pair, 1.00 * work(lm_head_pair_padded_rows(h->M), 256)},
                    {AJ_KERNEL_PAIR9, 9, pair, (rounds ? 1.03 + 140.0 / c.d_t : 1.06) * work(lm_head_pair9_padded_rows(h->M, 9), 288)},
                    {AJ_KERNEL_PAIR9, 7, rounds, 1.05 * work(lm_head_pair9_padded_rows(h->M, 7), 224)},
                    {AJ_KERNEL_PAIR9, 6, rounds, 1.085 * work(lm_head_pair9_padded_rows(h->M, 6), 192)},
                    {AJ_KERNEL_PAIR9, 5, rounds, 1.25 * work(lm_head_pair9_padded_rows(h->M, 5), 160)},
                    {AJ_KERNEL_BIG, 0, lm_head_mfma_supports(AJ_KERNEL_BIG, h->M, c.V, c.d_t),
                     1.10 * work(lm_head_mfma_padded_rows(AJ_KERNEL_BIG, h->M), 256)},
                    {AJ_KERNEL_TALL, 0, lm_head_mfma_supports(AJ_KERNEL_TALL, h->M, c.V, c.d_t),
                     (rounds ? 1.24 : 1.20) * work(tall, tall_rows)},
                };
                v = AJ_KERNEL_TILE;
                double best = 0.0;
                for (const auto &k : cand)
                    if (k.ok && (v == AJ_KERNEL_TILE || k.cost < best)) {
                        v = k.kernel;
                        h->row_blocks = k.row_blocks;
                        best = k.cost;
                    }
            }
        } else if (v == AJ_KERNEL_RESIDENT) {
            if (h->M > 0 && !lm_head_resident_supports(h->M, c.V, c.d_t, false)) return AJ_EINVAL;
        } else if (v == AJ_KERNEL_WIDE) {
            if (h->M > 0 && !lm_head_wide_supports(h->M, c.V, c.d_t, false)) return AJ_EINVAL;
        } else if (v == AJ_KERNEL_PAIR || v == AJ_KERNEL_PAIR9 ? (h->M > 0 && !lm_head_pair_supports(h->M, c.V, c.d_t))
                   : v != AJ_KERNEL_TILE && h->M > 0 && !lm_head_mfma_supports(v, h->M, c.V, c.d_t) &&
                         !(v == AJ_KERNEL_STREAM && lm_head_stream16_supports(h->M, c.V, c.d_t))) {
            return AJ_EINVAL;   // a forced variant that cannot run this shape
        }
        if (v == AJ_KERNEL_TILE && lm_head_tile_blocks(c.V) > 65535) return AJ_EINVAL;   // gridDim.y
        if ((c.flags & AJ_FLAG_FUSED_JUDGE) && h->M > 0) {
            // the fused judge row lives in the accumulator-resident kernel
            if (c.kernel != AJ_KERNEL_AUTO && c.kernel != AJ_KERNEL_RESIDENT) return AJ_EINVAL;
            if (!lm_head_resident_supports(h->M, c.V, c.d_t, false)) return AJ_EINVAL;
            v = AJ_KERNEL_RESIDENT;
        }
        h->variant = v;
        h->stream16 = v == AJ_KERNEL_STREAM && lm_head_stream16_supports(h->M, c.V, c.d_t);
        h->nblocks = v == AJ_KERNEL_TILE ? lm_head_tile_blocks(c.V)
                     : v == AJ_KERNEL_PAIR ? lm_head_pair_blocks(c.V)
                     : v == AJ_KERNEL_PAIR9 ? lm_head_pair9_blocks(c.V)
                     : v == AJ_KERNEL_RESIDENT ? lm_head_resident_blocks(c.V, h->num_cus)
                     : v == AJ_KERNEL_WIDE ? lm_head_wide_blocks(c.V)
                     : h->stream16     ? lm_head_stream16_blocks(c.V, h->num_cus)
                                       : lm_head_mfma_blocks(v, c.V, c.d_t, h->num_cus);
    }
    if (h->M > 0 && c.dtype == AJ_BF16 && c.kernel == AJ_KERNEL_AUTO && !(c.flags & AJ_FLAG_FUSED_JUDGE) && !h->stream16) {
        const SlabPlan p = slab_plan(h->M, c.V, c.d_t, h->fp8w, h->num_cus);
        if (two_row_tiles_win(h, p)) {
            h->variant = AJ_KERNEL_PAIR9;
            h->row_blocks = 5;
            h->nblocks = lm_head_pair9_blocks(c.V);
        } else if (slab_wins(h, p)) {
            h->slab = p.tile;
            // A k order of its own for every vocabulary tile spreads the streams over the memory channels (33 rows, d_t = 8192,
            // V = 32000: 77 us, 103 without; 48 x 4096 x 50257: 64, 85; sizes that are no power of two 0 .. 5 %) but gives equal W_lm
            // rows in different tiles sums that differ by rounding.  Only the accumulator-resident kernel does that too; the
            // others sum every row in one order, so that the lowest of equal rows wins, and so does what replaces them: there, where rows
            // are a multiple of 4096 bytes apart, one order that interleaves their halves, which gives most of it (86 us, 68; 122 x
            // 4096 x 32000 63.2 -> 61.1, 120 x 4096 x 72000 170 -> 166).  Several rounds of tiles at 4096 elements do better with that too: 99 x 4096 x 80000
            // rotated 154 us, interleaved 125, ascending 132; 33 x 4096 x 76000 100, 97, 114.  At 2048, 6144, 8192, 10240 and 12288 elements rotating
            // is 0 .. 2 % faster in several rounds too (geometric means of 6 .. 14 shapes each, 3 .. 99 rows, V 32000 .. 128256; 6 % in one round at 8192)
            const size_t row_bytes = (size_t)c.d_t * (h->fp8w ? 1 : 2);
            const bool even_rows = row_bytes % 4096 == 0;
            const bool rotate = h->variant == AJ_KERNEL_RESIDENT && !(p.rounds > 1 && c.d_t == 4096 && !h->fp8w);
            // A rotation by 5 slabs and tiles of 5 x 2^17 or 5 x 2^18 bytes (160 rows of 8192, 40 or 80 of 16384) meet on the memory channels again:
            // 9 instead (FP8, 30 x 8192 x 40796 91 -> 68 us, tiles 8 rows higher 71; 3 x 16384 x 19461 90 -> 81; bf16 8 x 8192 x 19969 80 -> 69).  Not
            // everywhere: over 11371 shapes 9, 13 or 1 take 1.00 .. 1.01 of the time of 5 on average, with such heights of their own
            const double tile_bytes = (double)p.tile.wv * p.tile.rows * row_bytes / (5 << 17);
            const bool meets = fabs(tile_bytes - 1.0) < 0.03 || fabs(tile_bytes - 2.0) < 0.06;
            h->slab.rot = rotate ? (meets ? 9 : 5) : even_rows && slab_interleaves(h->slab.wv, h->slab.mb, h->fp8w) ? INTERLEAVE : 0;
            h->variant = VARIANT_SLAB;
            h->nblocks = p.nblocks;
        }
    }
    return AJ_OK;
}

extern "C" int aj_create(const aj_config *cfg, aj_handle **out)
{
    if (out) *out = nullptr;
    if (!cfg || !out) return AJ_EINVAL;
    const aj_config &c = *cfg;
    aj_handle *h = new (std::nothrow) aj_handle();
    if (!h) return AJ_ENOMEM;
    const int rc = plan_handle(c, h);
    if (rc != AJ_OK) {
        delete h;
        return rc;
    }
    if (h->M > 0) {
        const size_t np = (size_t)h->nblocks * h->M;
        bool ok = hipMalloc(&h->part, np * sizeof(Best)) == hipSuccess &&
                  hipMalloc(&h->t_star, (size_t)h->M * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&h->maxlogit, (size_t)h->M * sizeof(float)) == hipSuccess &&
                  hipMalloc(&h->rej, (size_t)h->M) == hipSuccess;
        if (ok && (c.flags & AJ_FLAG_DEBUG))
            ok = hipMalloc(&h->score, (size_t)2 * c.B * c.K * sizeof(float)) == hipSuccess;
        if (ok && (c.flags & AJ_FLAG_FUSED_JUDGE))
            ok = hipMalloc(&h->zt, (size_t)h->M * sizeof(float)) == hipSuccess;
        if (ok && (c.flags & AJ_FLAG_TOPK))
            ok = hipMalloc(&h->cnt, np * sizeof(int32_t)) == hipSuccess &&
                 hipMalloc(&h->thr, (size_t)h->M * sizeof(float)) == hipSuccess &&
                 hipMalloc(&h->thr_tok, (size_t)h->M * sizeof(int32_t)) == hipSuccess &&
                 hipMalloc(&h->rank, (size_t)h->M * sizeof(int32_t)) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            free_all(h);
            delete h;
            return AJ_ENOMEM;
        }
    }
    if (c.flags & AJ_FLAG_PROFILE) {
        h->ev_ok = true;
        for (int i = 0; i < 64; ++i)
            for (int j = 0; j < 2; ++j) {
                const hipError_t e = hipEventCreate(&h->ev[i][j]);
                if (e != hipSuccess) {   // destroy what exists, then fail
                    for (int ii = 0; ii <= i; ++ii)
                        for (int jj = 0; jj < (ii == i ? j : 2); ++jj) (void)hipEventDestroy(h->ev[ii][jj]);
                    h->ev_ok = false;
                    free_all(h);
                    delete h;
                    return hip_fail(e);
                }
            }
    }
    *out = h;
    return AJ_OK;
}

extern "C" int aj_destroy(aj_handle *h)
{
    if (!h) return AJ_EINVAL;
    free_all(h);
    delete h;
    return AJ_OK;
}

static hipError_t launch_lm_head(aj_handle *h, const void *hidden_t, const void *W_lm, float *dump, hipStream_t s,
                                 bool topk = false, const uint64_t *key = nullptr, float inv_temp = 1.f,
                                 const void *judge_w = nullptr)
{
    LmHeadArgs a;
    a.H = hidden_t;
    a.W = W_lm;
    a.M = h->M;
    a.V = h->cfg.V;
    a.d = h->cfg.d_t;
    a.part = h->part;
    a.nblocks = h->nblocks;
    a.dump = dump;
    a.thr = topk ? h->thr : nullptr;
    a.thr_tok = topk ? h->thr_tok : nullptr;
    a.cnt = topk ? h->cnt : nullptr;
    a.key = key;
    a.inv_temp = inv_temp;
    a.judge_w = judge_w;
    a.zt = judge_w ? h->zt : nullptr;
    if (h->variant == -1) return lm_head_f32(a, h->num_cus, s);
    if (h->variant == VARIANT_F32_SPLIT) return lm_head_f32_split(h->split, a, s);
    if (h->variant == VARIANT_SLAB) return h->fp8w ? lm_head_slab_fp8w(h->slab, a, s) : lm_head_slab_bf16(h->slab, a, s);
    if (h->variant == AJ_KERNEL_TILE) return lm_head_tile_bf16(a, s);
    if (h->variant == AJ_KERNEL_RESIDENT)
        return h->fp8w ? lm_head_resident_fp8w(a, h->num_cus, s) : lm_head_resident_bf16(a, h->num_cus, s);
    if (h->variant == AJ_KERNEL_WIDE) return h->fp8w ? lm_head_wide_fp8w(a, h->num_cus, s) : lm_head_wide_bf16(a, h->num_cus, s);
    if (h->fp8w) return lm_head_stream16_fp8w(a, h->num_cus, s);
    if (h->stream16) return lm_head_stream16_bf16(a, h->num_cus, s);
    if (h->variant == AJ_KERNEL_PAIR) return lm_head_pair_bf16(a, h->num_cus, s);
    if (h->variant == AJ_KERNEL_PAIR9) return lm_head_pair9_bf16(h->row_blocks, a, h->num_cus, s);
    return lm_head_mfma_bf16(h->variant, a, h->num_cus, s);
}

// aj_verify, aj_verify_sampled and aj_verify_tree: the same steps; key == nullptr selects the greedy token,
// parent == nullptr a chain of draft tokens
static int verify_common(aj_handle *h, const void *hidden_t, const void *hidden_d, const void *W_lm,
                         const int32_t *draft_tok, const void *clf_w, float clf_b, float tau,
                         const uint64_t *key, float inv_temp, const int32_t *parent, int32_t *out_node,
                         int32_t *out_len, int32_t *out_tok, void *stream)
{
    if (!h) return AJ_EINVAL;
    if (!(tau >= 0.f && tau <= 1.f)) return AJ_EINVAL;   // also refuses NaN
    if (!isfinite(clf_b)) return AJ_EINVAL;
    if (h->M == 0) return AJ_OK;
    const aj_config &c = h->cfg;
    if (!hidden_t || !W_lm || !draft_tok || !clf_w || !out_len || !out_tok) return AJ_EINVAL;
    if (c.d_d > 0 && !hidden_d) return AJ_EINVAL;
    if (!aligned16(hidden_t) || !aligned16(W_lm) || !aligned16(clf_w) || (c.d_d > 0 && !aligned16(hidden_d)))
        return AJ_EINVAL;
    hipStream_t s = (hipStream_t)stream;

    const bool prof = h->ev_ok;
    const int slot = (int)(h->calls % 64);
    hipError_t e;
    if (prof && (e = hipEventRecord(h->ev[slot][0], s)) != hipSuccess) return hip_fail(e);
    // fused judge row: greedy chains and trees on a handle created for it (the sampling variant computes the judge
    // in the tail, as usual)
    const bool fused = h->zt && !key && h->variant == AJ_KERNEL_RESIDENT && !h->fp8w;
    if ((e = launch_lm_head(h, hidden_t, W_lm, nullptr, s, false, key, inv_temp, fused ? clf_w : nullptr)) != hipSuccess)
        return hip_fail(e);
    if (prof && (e = hipEventRecord(h->ev[slot][1], s)) != hipSuccess) return hip_fail(e);
    if (prof) h->calls++;

    TailArgs t;
    t.hidden_t = hidden_t;
    t.hidden_d = hidden_d;
    t.clf_w = clf_w;
    t.draft_tok = draft_tok;
    t.part = h->part;
    t.nblocks = h->nblocks;
    t.B = c.B;
    t.K = c.K;
    t.d_t = c.d_t;
    t.d_d = c.d_d;
    t.V = c.V;
    t.dtype = c.dtype;
    t.feat_offset = c.feat_offset;
    t.clf_b = clf_b;
    // threshold in logit space, computed in double from the float tau, rounded once to float
    t.zthr = tau <= 0.f ? -INFINITY : (tau >= 1.f ? INFINITY : (float)log((double)tau / (1.0 - (double)tau)));
    t.t_star = h->t_star;
    t.maxlogit = h->maxlogit;
    t.zt = fused ? h->zt : nullptr;
    t.score = h->score;
    t.rej = h->rej;
    t.out_len = out_len;
    t.out_tok = out_tok;
    t.parent = parent;
    t.out_node = out_node;
    if ((e = verify_tail(t, s)) != hipSuccess) return hip_fail(e);
    return AJ_OK;
}

extern "C" int aj_verify(aj_handle *h, const void *hidden_t, const void *hidden_d, const void *W_lm,
                         const int32_t *draft_tok, const void *clf_w, float clf_b, float tau,
                         int32_t *out_len, int32_t *out_tok, void *stream)
{
    return verify_common(h, hidden_t, hidden_d, W_lm, draft_tok, clf_w, clf_b, tau, nullptr, 1.f, nullptr, nullptr,
                         out_len, out_tok, stream);
}

// ---- aj_verify without any allocation: the workspace is a static device array -----------------------------
// Every GPU the library runs on holds its own copy of `scratch` at its own address until the process ends.  In
// host code the array's NAME is only a stand-in: the device address comes from hipGetSymbolAddress, once per
// device with that device current, and that pointer is what kernels get.
static __device__ __align__(256) unsigned char scratch[AJ_STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[MAX_DEVICES];   // device address of `scratch` per device, nullptr until first use

static int scratch_of_current_device(int device, unsigned char **out)
{
    if (device < 0 || device >= MAX_DEVICES) return AJ_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (!p) return hip_fail(hipErrorInvalidSymbol);
        g_scratch_ptr[device] = p;
    }
    *out = (unsigned char *)g_scratch_ptr[device];
    return AJ_OK;
}

static size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }

extern "C" int aj_verify_static(const aj_config *cfg, const void *hidden_t, const void *hidden_d, const void *W_lm,
                                const int32_t *draft_tok, const void *clf_w, float clf_b, float tau,
                                int32_t *out_len, int32_t *out_tok, void *stream)
{
    if (!cfg) return AJ_EINVAL;
    if (cfg->flags != 0) return AJ_EINVAL;        // debug scores, profiling events and top-K counts need a handle
    aj_handle h = {};
    const int rc = plan_handle(*cfg, &h);          // validates, chooses the kernel; allocates nothing
    if (rc != AJ_OK) return rc;
    if (h.M == 0) return AJ_OK;
    // workspace of this shape: [M][nblocks] partials, then t_star[M], maxlogit[M] and the rejected-slot flags
    // (M bytes), each 256-byte aligned
    // (fp32: of the partials of the fp32 kernel's tiles, the smaller ones, whichever kernel runs: what the entry point takes does not
    // hang on a cost table)
    const int limit_blocks = h.variant == VARIANT_F32_SPLIT ? lm_head_f32_blocks(h.M, cfg->V, cfg->d_t, h.num_cus) : h.nblocks;
    const size_t part_bytes = round256((size_t)h.M * limit_blocks * sizeof(Best));
    const size_t row_bytes = round256((size_t)h.M * sizeof(int32_t));
    if (part_bytes + 3 * row_bytes > AJ_STATIC_SCRATCH_BYTES) return AJ_ELIMIT;
    unsigned char *base = nullptr;
    const int rs = scratch_of_current_device(h.device, &base);
    if (rs != AJ_OK) return rs;
    // every word the tail kernel reads is written by the LM-head kernel of the same call (one partial per row and
    // block, empty blocks included), so nothing has to start at zero and the last call's contents do not matter
    h.part = (Best *)base;
    h.t_star = (int32_t *)(base + part_bytes);
    h.maxlogit = (float *)(base + part_bytes + row_bytes);
    h.rej = base + part_bytes + 2 * row_bytes;
    return verify_common(&h, hidden_t, hidden_d, W_lm, draft_tok, clf_w, clf_b, tau, nullptr, 1.f, nullptr, nullptr,
                         out_len, out_tok, stream);
}

extern "C" int aj_verify_tree(aj_handle *h, const void *hidden_t, const void *hidden_d, const void *W_lm,
                              const int32_t *draft_tok, const int32_t *parent, const void *clf_w, float clf_b,
                              float tau, int32_t *out_len, int32_t *out_tok, int32_t *out_node, void *stream)
{
    if (!h) return AJ_EINVAL;
    if (h->M > 0 && (!parent || !out_node)) return AJ_EINVAL;
    return verify_common(h, hidden_t, hidden_d, W_lm, draft_tok, clf_w, clf_b, tau, nullptr, 1.f, parent, out_node,
                         out_len, out_tok, stream);
}

extern "C" int aj_verify_sampled(aj_handle *h, const void *hidden_t, const void *hidden_d, const void *W_lm,
                                 const int32_t *draft_tok, const void *clf_w, float clf_b, float tau,
                                 float inv_temperature, const uint64_t *row_key,
                                 int32_t *out_len, int32_t *out_tok, void *stream)
{
    if (!h) return AJ_EINVAL;
    if (!(inv_temperature >= 0.f) || !isfinite(inv_temperature)) return AJ_EINVAL;
    if (h->M > 0 && (!row_key || (((uintptr_t)row_key) & 7u))) return AJ_EINVAL;
    return verify_common(h, hidden_t, hidden_d, W_lm, draft_tok, clf_w, clf_b, tau, row_key, inv_temperature, nullptr,
                         nullptr, out_len, out_tok, stream);
}

extern "C" int aj_verify_topk(aj_handle *h, const void *hidden_t, const void *W_lm, const int32_t *draft_tok,
                              int32_t top_k, int32_t *out_len, int32_t *out_tok, void *stream)
{
    if (!h) return AJ_EINVAL;
    if (top_k < 1) return AJ_EINVAL;
    if (!(h->cfg.flags & AJ_FLAG_TOPK)) return AJ_ESTATE;
    if (h->M == 0) return AJ_OK;
    const aj_config &c = h->cfg;
    if (!hidden_t || !W_lm || !draft_tok || !out_len || !out_tok) return AJ_EINVAL;
    if (!aligned16(hidden_t) || !aligned16(W_lm)) return AJ_EINVAL;
    hipStream_t s = (hipStream_t)stream;

    TopkArgs t;
    t.hidden_t = hidden_t;
    t.W_lm = W_lm;
    t.draft_tok = draft_tok;
    t.B = c.B;
    t.K = c.K;
    t.d_t = c.d_t;
    t.V = c.V;
    t.dtype = c.dtype;
    t.top_k = top_k;
    t.thr = h->thr;
    t.thr_tok = h->thr_tok;
    t.part = h->part;
    t.cnt = h->cnt;
    t.nblocks = h->nblocks;
    t.t_star = h->t_star;
    t.maxlogit = h->maxlogit;
    t.rank = h->rank;
    t.out_len = out_len;
    t.out_tok = out_tok;

    hipError_t e;
    if ((e = topk_draft_logit(t, s)) != hipSuccess) return hip_fail(e);
    const bool prof = h->ev_ok;
    const int slot = (int)(h->calls % 64);
    if (prof && (e = hipEventRecord(h->ev[slot][0], s)) != hipSuccess) return hip_fail(e);
    if ((e = launch_lm_head(h, hidden_t, W_lm, nullptr, s, true)) != hipSuccess) return hip_fail(e);
    if (prof && (e = hipEventRecord(h->ev[slot][1], s)) != hipSuccess) return hip_fail(e);
    if (prof) h->calls++;
    if ((e = topk_tail(t, s)) != hipSuccess) return hip_fail(e);
    return AJ_OK;
}

extern "C" int aj_debug_copy_rank(aj_handle *h, int32_t *rank_host, void *stream)
{
    if (!h || !rank_host) return AJ_EINVAL;
    if (!(h->cfg.flags & AJ_FLAG_TOPK)) return AJ_ESTATE;
    if (h->M == 0) return AJ_OK;
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e == hipSuccess) e = hipMemcpy(rank_host, h->rank, (size_t)h->M * sizeof(int32_t), hipMemcpyDeviceToHost);
    return e == hipSuccess ? AJ_OK : hip_fail(e);
}

extern "C" int aj_debug_ptrs(aj_handle *h, const int32_t **t_star, const float **maxlogit, const float **score)
{
    if (!h) return AJ_EINVAL;
    if (score && !h->score && h->M > 0) return AJ_ESTATE;
    if (t_star) *t_star = h->t_star;
    if (maxlogit) *maxlogit = h->maxlogit;
    if (score) *score = h->score;
    return AJ_OK;
}

extern "C" int aj_debug_copy(aj_handle *h, int32_t *t_star_host, float *maxlogit_host, float *score_host,
                             void *stream)
{
    if (!h) return AJ_EINVAL;
    if (score_host && !h->score && h->M > 0) return AJ_ESTATE;
    if (h->M == 0) return AJ_OK;
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e == hipSuccess && t_star_host)
        e = hipMemcpy(t_star_host, h->t_star, (size_t)h->M * sizeof(int32_t), hipMemcpyDeviceToHost);
    if (e == hipSuccess && maxlogit_host)
        e = hipMemcpy(maxlogit_host, h->maxlogit, (size_t)h->M * sizeof(float), hipMemcpyDeviceToHost);
    if (e == hipSuccess && score_host)
        e = hipMemcpy(score_host, h->score, (size_t)2 * h->cfg.B * h->cfg.K * sizeof(float), hipMemcpyDeviceToHost);
    return e == hipSuccess ? AJ_OK : hip_fail(e);
}

extern "C" int aj_debug_logits(aj_handle *h, const void *hidden_t, const void *W_lm, float *logits, void *stream)
{
    if (!h) return AJ_EINVAL;
    if (h->M == 0) return AJ_OK;
    if (!hidden_t || !W_lm || !logits || !aligned16(hidden_t) || !aligned16(W_lm)) return AJ_EINVAL;
    hipError_t e = launch_lm_head(h, hidden_t, W_lm, logits, (hipStream_t)stream);
    return e == hipSuccess ? AJ_OK : hip_fail(e);
}

extern "C" int aj_profile_read(aj_handle *h, float *ms, int32_t *n)
{
    if (!h || !ms || !n || *n < 0) return AJ_EINVAL;
    if (!h->ev_ok) return AJ_ESTATE;
    const uint64_t have = h->calls < 64 ? h->calls : 64;
    const int want = (int)((uint64_t)*n < have ? (uint64_t)*n : have);
    for (int i = 0; i < want; ++i) {
        const int slot = (int)((h->calls - want + i) % 64);
        hipError_t e = hipEventSynchronize(h->ev[slot][1]);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms[i], h->ev[slot][0], h->ev[slot][1]);
        if (e != hipSuccess) return hip_fail(e);
    }
    *n = want;
    return AJ_OK;
}

extern "C" int aj_debug_tile(const aj_handle *h, int32_t *vocab_rows, int32_t *verify_rows)
{
    if (!h || !vocab_rows || !verify_rows) return AJ_EINVAL;
    if (h->M == 0) return AJ_ESTATE;
    if (h->variant == VARIANT_SLAB) {
        *vocab_rows = h->slab.wv * h->slab.rows;
        *verify_rows = 16 * h->slab.mb;
        return AJ_OK;
    }
    if (h->variant == VARIANT_F32_SPLIT) {
        *vocab_rows = 16 * h->split.wv * h->split.nb;
        *verify_rows = 16 * h->split.mb;
        return AJ_OK;
    }
    if (h->variant != -1) return AJ_ESTATE;
    lm_head_f32_tile(h->M, h->cfg.V, h->cfg.d_t, h->num_cus, vocab_rows, verify_rows);
    return AJ_OK;
}

extern "C" int aj_debug_form(const aj_handle *h, int32_t *waves, int32_t *vocab_blocks, int32_t *k_order)
{
    if (!h || !waves || !vocab_blocks || !k_order) return AJ_EINVAL;
    if (h->M == 0) return AJ_ESTATE;
    if (h->variant == VARIANT_SLAB) {
        *waves = h->slab.wv;
        *vocab_blocks = 4 * h->slab.nb / h->slab.wv;
        *k_order = h->slab.rot == INTERLEAVE ? 1 : h->slab.rot ? 2 : 0;
        return AJ_OK;
    }
    if (h->variant != VARIANT_F32_SPLIT) return AJ_ESTATE;
    *waves = h->split.wv;
    *vocab_blocks = h->split.nb;
    *k_order = h->cfg.d_t % 1024 == 0;
    return AJ_OK;
}

extern "C" const char *aj_kernel_name(const aj_handle *h)
{
    if (!h) return "none";
    switch (h->variant) {
        case -1: return "lm_head_f32";
        case VARIANT_F32_SPLIT: return "lm_head_f32_split";
        case VARIANT_SLAB: return h->fp8w ? "lm_head_slab_fp8w" : "lm_head_slab_bf16";
        case AJ_KERNEL_TILE: return "lm_head_tile_bf16";
        case AJ_KERNEL_STREAM:
            return h->fp8w ? "lm_head_stream16_fp8w" : h->stream16 ? "lm_head_stream16_bf16" : "lm_head_stream_bf16";
        case AJ_KERNEL_BIG: return "lm_head_big_bf16";
        case AJ_KERNEL_TALL: return "lm_head_tall_bf16";
        case AJ_KERNEL_PAIR: return "lm_head_pair_bf16";
        case AJ_KERNEL_PAIR9: {
            static const char *const name[5] = {"lm_head_pair5_bf16", "lm_head_pair6_bf16", "lm_head_pair7_bf16", "",
                                                "lm_head_pair9_bf16"};
            return name[h->row_blocks - 5];
        }
        case AJ_KERNEL_WIDE: return h->fp8w ? "lm_head_wide_fp8w" : "lm_head_wide_bf16";
        case AJ_KERNEL_RESIDENT: return h->fp8w ? "lm_head_resident_fp8w" : "lm_head_resident_bf16";
        default: return "unknown";
    }
}
