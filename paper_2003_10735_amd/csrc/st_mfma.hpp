// Vector types and operand layouts of the gfx950 matrix-core builtins.
#pragma once
#include "st_common.hpp"

namespace st {
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// v_mfma_f32_32x32x16_bf16: D[32x32] += A[32x16] * B[16x32].  Lane l supplies A[l % 32][8*(l/32) .. +7]
// and B[8*(l/32) .. +7][l % 32]; it receives D[8*(r/4) + 4*(l/32) + r%4][l % 32] in register r.

// Stores at device scope (sc1): they go through the L2 cache to memory as they are made, `off` bytes behind `base`, which is the same for all
// lanes.  A plain store stays in L2 as a dirty line until its launch ends, and the next launch waits for the write-back: 7.9 MB written by
// 240 blocks and nothing else 2.83 us a launch, through the cache 2.32.  The reader fetches the data from memory either way (what a step
// moves turns every L2 over between a write and its read).  For whole 128-byte lines of outputs that are large: the logits' shares, rows of
// 80 bytes in pieces of 16, are dearer this way (4 x 90 x 160 cells 7524 -> 7610 us a call), and where everything a step writes stays in L2 a
// plain store is the cheaper one (weight gradients of 16 x 16 cells, float32: a call 192 -> 196 us).
// Plain -> this, us a call: key frame at 90 x 160 cells 608 -> 585, at 135 x 240 1171 -> 1137, 4 x 90 x 160 cells, 320 -> 256 -> 256 channels
// 7483 -> 7410, 60 x 107 cells, 96 -> 48 -> 48 channels 208.7 -> 204.9; calls of four steps at 45 x 80 cells 222.5 -> 218.1 with 128 channels and
// 188.3 -> 187.5 with 64.  Below that the bfloat16 kernels lose a little by it: 64 channels at 30 x 53 cells 168.5 -> 169.8, 23 x 40 154.7 -> 156.6,
// 16 x 24 147.4 -> 150.2 (128 channels 169.1 -> 170.0, 256 228.5 -> 228.1).  They have no line by size for it: with plain stores of convolution
// outputs and classifier gradients of a megabyte or less 16 x 24 cells took 147.7 instead of 148.9, but 43 x 78 with 128 channels 204 instead
// of 201, and asking for the size in the classifier's backward cost the large grids (135 x 240 cells, four steps 715 -> 719.5).
__device__ __forceinline__ void store_through(void* base, unsigned off, u32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000), (int)off, 0, 16);
}
__device__ __forceinline__ void store_through(void* base, unsigned off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000), (int)off, 0, 16);
}

// Channel-major operand copies ("XT") feed the weight-gradient kernels, whose MFMA fragments are
// 32 channels x 8 consecutive positions.  They are stored blocked so that such a fragment is one
// contiguous 512-byte run and a wavefront's fragment load is fully coalesced:
//     [channel / 32][column / 8][channel % 32][column % 8],   column = guard + padded position,
// with NG = PPT / 8 column groups per channel block.
__host__ __device__ __forceinline__ size_t xt_index(int c, int col, int NG)
{
    return (((size_t)(c >> 5) * NG + (col >> 3)) << 8) + ((c & 31) << 3) + (col & 7);
}

// Weights of the 3x3 matrix-core convolutions, [rows][9 taps][K], are kept in the order in which
// that kernel's wavefronts consume them: one A fragment (32 rows x 16 k of one tap, lane l holding
// row l % 32, k 8*(l/32) .. +7) is one contiguous 1 KB run,
//     [row / 32][tap][k / 16][(k / 8) % 2][row % 32][k % 8],
// in other words [row / 32][tap][k / 8][row % 32][k % 8], which also serves a K that ends with half a fragment.
__host__ __device__ __forceinline__ size_t wfrag_index(int row, int tap, int k, int K)
{
    return ((((size_t)(row >> 5) * 9 + tap) * (K >> 3) + (k >> 3)) * 32 + (row & 31)) * 8 + (k & 7);
}

// Float32 path: activations in runs of eight channels, [c / 8][column][8], column = guard + padded position, PPT
// columns per run.
__host__ __device__ __forceinline__ size_t pos8_index(int c, int col, int PPT) { return ((size_t)(c >> 3) * PPT + col) * 8 + (c & 7); }

// Its 3x3 weights lie in the order of wfrag_index too, as float32, where operands are split times F32_SPLIT_SCALE: the factor that
// either operand of a split product has (k_conv_f32.hip says why).  F32_SPLIT_BACK takes both back out of a sum.
constexpr float F32_SPLIT_SCALE = 0x1p24f, F32_SPLIT_BACK = 0x1p-48f;

// v_mfma_f32_32x32x2_f32 (the float32 path's classifier): lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32]; D as above.
// W3 for its backward, K (a multiple of eight) classes per row: the A operands of four MFMAs (32 rows x 8 k, lane l holding
// row l % 32, k 4*(l/32) .. +3) are one contiguous 1 KB run,  [row / 32][k / 8][(k / 4) % 2][row % 32][k % 4].
__host__ __device__ __forceinline__ size_t wfrag32_index(int row, int k, int K)
{
    return (((size_t)(row >> 5) * (K >> 3) + (k >> 3)) * 64 + ((k >> 2) & 1) * 32 + (row & 31)) * 4 + (k & 3);
}
}  // namespace st
