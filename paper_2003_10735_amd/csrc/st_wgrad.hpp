// Closing part of the weight-gradient kernels: the four wavefronts of a block add their 32 x 32 x 9
// blocks through LDS and store the sum.
#pragma once
#include "st_mfma.hpp"

namespace st {

// LDS of those kernels: four blocks [9 taps * 32 o][32 i], and [4][32] sums for the bias gradient
constexpr size_t WGRAD_SMEM_BYTES = (size_t)(4 * 9 * 32 * 32 + 4 * 32) * sizeof(float);

// Every wavefront leaves its block in LDS as [tap][o][i]; then all 256 threads add the four copies in the
// order ((w0 + w1) + w2) + w3 and write the result with 16-byte stores.  X is the MFMA's A operand,
// so a lane holds four consecutive input channels i of one output channel o per register group: one
// 16-byte LDS write.  Rows are 128 bytes; the 16-byte chunk c of row o is stored at chunk
// c ^ ((o >> 1) & 7), which spreads the 16 lanes of a write (and of a read) over all banks.
// acc[0..8]: the taps.  dW: [cout][9][cin] of this split.  (A tile's 32-bit offsets: a whole one has 32 output channels, so that a row of
// 9 cin floats is below 2^25 bytes.)  THROUGH: past the caches (store_through).
template <bool THROUGH, int N>
__device__ __forceinline__ void wgrad_reduce_store(const f32x16 (&acc)[N], float* red, float* dW, int o0, int i0, int cout, int cin)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int sw = (l32 >> 1) & 7;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const f32x4 v = {acc[t][gq * 4], acc[t][gq * 4 + 1], acc[t][gq * 4 + 2], acc[t][gq * 4 + 3]};
            *(f32x4*)(red + ((wave * 9 + t) * 32 + l32) * 32 + (((gq * 2 + lhi) ^ sw) << 2)) = v;
        }
    __syncthreads();
    auto sum_of = [&](int q) {
        const int row = q >> 3, part = q & 7;
        const int chunk = (part ^ (((row & 31) >> 1) & 7)) << 2;
        const f32x4 v0 = *(const f32x4*)(red + ((0 * 9 * 32 + row) * 32 + chunk));
        const f32x4 v1 = *(const f32x4*)(red + ((1 * 9 * 32 + row) * 32 + chunk));
        const f32x4 v2 = *(const f32x4*)(red + ((2 * 9 * 32 + row) * 32 + chunk));
        const f32x4 v3 = *(const f32x4*)(red + ((3 * 9 * 32 + row) * 32 + chunk));
        return ((v0 + v1) + v2) + v3;
    };
    auto place_of = [&](int q) {
        const int t = q >> 8, ol = (q >> 3) & 31, part = q & 7;
        return dW + ((size_t)(o0 + ol) * 9 + t) * cin + i0 + part * 4;
    };
    auto offset_of = [&](int q) { return (unsigned)((((q >> 3) & 31) * 9 + (q >> 8)) * cin + (q & 7) * 4) * 4u; };
    if (o0 + 32 <= cout && i0 + 32 <= cin && ((cin | (int)((uintptr_t)dW >> 2)) & 3) == 0) {
        for (int q = tid; q < 9 * 32 * 8; q += 256) {
            if (THROUGH) store_through(dW + (size_t)o0 * 9 * cin + i0, offset_of(q), __builtin_bit_cast(u32x4, sum_of(q)));
            else *(f32x4*)place_of(q) = sum_of(q);
        }
    } else {
        // a tile with padded channels of a narrow head: those have no gradient to store
        for (int q = tid; q < 9 * 32 * 8; q += 256) {
            const f32x4 sum = sum_of(q);
            float* dst = place_of(q);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (o0 + ((q >> 3) & 31) < cout && i0 + (q & 7) * 4 + e < cin) dst[e] = sum[e];
        }
    }
}

}  // namespace st
