// Dot product of two rows by a wave, for the small kernels around the LM head.
#pragma once
#include "aj_internal.h"

namespace aj {

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// wave-wide partial dot of n elements (n % 8 == 0 for bf16, % 4 for f32), fp32 accumulation.
// Four 16-byte chunks per operand are requested before any is used: this kernel is a chain of
// memory round trips, so what counts is how many loads are in flight, not the arithmetic.
template <bool BF16, int U = 4>
__device__ __forceinline__ float dot_part(const void *x, const void *w, int n, int lane)
{
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.f;
    const int nchunks = n / (BF16 ? 8 : 4);
    const u32x4 *xp = (const u32x4 *)x, *wp = (const u32x4 *)w;
    for (int c0 = lane; c0 < nchunks; c0 += 64 * U) {
        u32x4 xv[U], wv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 64 * u;
            const bool in = c < nchunks;
            xv[u] = in ? xp[c] : u32x4{0, 0, 0, 0};
            wv[u] = in ? wp[c] : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (BF16) {
                    acc[u] = fmaf(bf16_lo(xv[u][q]), bf16_lo(wv[u][q]), acc[u]);
                    acc[u] = fmaf(bf16_hi(xv[u][q]), bf16_hi(wv[u][q]), acc[u]);
                } else {
                    acc[u] = fmaf(__uint_as_float(xv[u][q]), __uint_as_float(wv[u][q]), acc[u]);
                }
            }
        }
    }
    if constexpr (U == 1) return acc[0];
    else {
        float sum = 0.f;
#pragma unroll
        for (int u = 0; u < U; u += 4) sum += (acc[u] + acc[u + 1]) + (acc[u + 2] + acc[u + 3]);
        return sum;
    }
}

}  // namespace aj
