// Work that opens a call -- packing the features, the label-dependent half of the gradient --
// written as per-block device functions, so that it can run either as kernels of its own or as
// roles of the one launch that opens a call (k_call_begin, next to the optimiser kernel).
#pragma once
#include "st_kernels.hpp"
#include "st_mfma.hpp"

namespace st {

// Float32 path: features [n, c_in, h, w] (or [n, h, w, c_in]: Geo::nhwc) -> runs of eight channels
// (pos8_index), the whole padded grid (zeros on the border and in padded channels).  One thread per
// padded position and run: position tile bx (256 positions), run by.
template <class Tin>
__device__ __forceinline__ void pack_features_f32_block(const Tin* __restrict__ f, float* __restrict__ out, const Geo& g, int PPT,
                                                        int guard, int bx, int by)
{
    const int mp = bx * 256 + threadIdx.x, frame = g.Hp * g.Wp, c0 = by * 8;
    if (mp >= g.padded_positions()) return;
    const int img = mp / frame, rr = mp - img * frame, y = rr / g.Wp - 1, x = rr % g.Wp - 1;
    const bool inside = y >= 0 && y < g.h && x >= 0 && x < g.w;
    const size_t at = !inside ? 0 : g.nhwc ? (((size_t)img * g.h + y) * g.w + x) * g.c_in : (size_t)img * g.c_in * g.h * g.w + y * g.w + x;
    const size_t step = g.nhwc ? 1 : (size_t)g.h * g.w;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = inside && c0 + e < g.c_in ? to_f32(f[at + (c0 + e) * step]) : 0.f;
    float4* dst = (float4*)(out + pos8_index(c0, guard + mp, PPT));
    dst[0] = make_float4(v[0], v[1], v[2], v[3]);
    dst[1] = make_float4(v[4], v[5], v[6], v[7]);
}

// bfloat16 path: features (Tin) -> padded position-major [n, Hp, Wp, ki] and, when
// outT != nullptr, a channel-major copy in the blocked layout of xt_index() for the
// weight-gradient kernel; the whole padded grid (zeros on the border and in padded channels).
// One block (256 threads) takes 64 padded positions (position tile bx) x 64 channels (by) through LDS, so that
// the reads (along x, or along c for Geo::nhwc) are contiguous and the writes are 16 bytes each.
// `tile` is 64 rows of PACKV_PITCH bfloat16 in LDS.
constexpr int PACKV_PITCH = 64 + 8;
template <class Tin>
__device__ __forceinline__ void pack_features_block(const Tin* __restrict__ f, bf16* __restrict__ out,
                                                    bf16* __restrict__ outT, const Geo& g, int PPT, int guard,
                                                    int bx, int by, bf16* tile)
{
    const int tid = threadIdx.x, mp0 = bx * 64, c0 = by * 64;
    const int frame = g.Hp * g.Wp, hw = g.h * g.w, PP = g.padded_positions();
    // cell (row-major over all frames) of padded position mp, or -1 on the border and behind the grid
    auto cell_of = [&](int mp) {
        const int img = mp / frame, rr = mp - img * frame, yp = rr / g.Wp, x = rr - yp * g.Wp - 1, y = yp - 1;
        return mp < PP && y >= 0 && y < g.h && x >= 0 && x < g.w ? img * hw + y * g.w + x : -1;
    };
    if (g.nhwc) {
        // eight channels of a position per thread: they go straight to the position-major copy
        const bool vec = g.c_in % 8 == 0 && ((uintptr_t)f & 15) == 0;
        bf16x8 o[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int i = tid + r * 256, pl = i >> 3, c = c0 + (i & 7) * 8;
            const int cell = cell_of(mp0 + pl);
            const Tin* src = f + (size_t)max(cell, 0) * g.c_in + c;
            if (vec) {
                typedef Tin tin8 __attribute__((ext_vector_type(8)));
                tin8 v = {};
                if (cell >= 0 && c < g.c_in) v = *(const tin8*)src;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[r][e] = from_f32<bf16>(to_f32(v[e]));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) o[r][e] = cell >= 0 && c + e < g.c_in ? from_f32<bf16>(to_f32(src[e])) : (bf16)0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int i = tid + r * 256, pl = i >> 3, cl = (i & 7) * 8;
            if (mp0 + pl < PP) *(bf16x8*)(out + (size_t)(mp0 + pl) * g.ki + c0 + cl) = o[r];
            if (outT)
#pragma unroll
                for (int e = 0; e < 8; ++e) tile[(cl + e) * PACKV_PITCH + pl] = o[r][e];
        }
        if (!outT) return;
        __syncthreads();
    } else {
        const int pl = tid & 63, cell = cell_of(mp0 + pl);
        const int img = max(cell, 0) / hw;
        const Tin* src = f + ((size_t)img * g.c_in + c0) * hw + (max(cell, 0) - img * hw);
        Tin v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int q = (tid >> 6) + 4 * k;
            v[k] = cell >= 0 && c0 + q < g.c_in ? src[(size_t)q * hw] : (Tin)0.f;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) tile[((tid >> 6) + 4 * k) * PACKV_PITCH + pl] = from_f32<bf16>(to_f32(v[k]));
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            // position-major: 8 channels of one position
            const int i = tid + r * 256, p = i >> 3, cq = i & 7;
            if (mp0 + p < PP) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = tile[(cq * 8 + e) * PACKV_PITCH + p];
                *(bf16x8*)(out + (size_t)(mp0 + p) * g.ki + c0 + cq * 8) = o;
            }
        }
        if (!outT) return;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        // channel-major: 8 positions of one channel (PP is a multiple of eight)
        const int i = tid + r * 256, ch = i >> 3, g8 = i & 7;
        if (mp0 + 8 * g8 < PP)
            *(bf16x8*)(outT + xt_index(c0 + ch, guard + mp0 + 8 * g8, PPT / 8)) = *(const bf16x8*)(tile + ch * PACKV_PITCH + 8 * g8);
    }
}

// The same for bfloat16 features with 16-byte reads (pack_vectors): one padded row yp (bz = img * Hp + yp),
// 64 channels (by), 64 padded columns xp0 .. xp0 + 63 (bx) per block.
__device__ __forceinline__ void pack_features_vec_block(const bf16* __restrict__ f, bf16* __restrict__ out,
                                                        bf16* __restrict__ outT, const Geo& g, int PPT, int guard,
                                                        int bx, int by, int bz, bf16* tile)
{
    const int xp0 = bx * 64, c0 = by * 64;
    const int img = bz / g.Hp, yp = bz % g.Hp;
    const bool row_in = yp >= 1 && yp <= g.h;
    const int tid = threadIdx.x;
    // source chunks of 8 columns x = 8q .. 8q + 7 land at padded columns x + 1; the tile's first
    // padded column (a border or an x = 8k - 1) comes from the chunk before
    bf16x8 v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = tid + r * 256, ch = i >> 3, q = i & 7;
        const int x = xp0 + 8 * q;                         // first column of the chunk
        v[r] = bf16x8{(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
        if (row_in && x < g.w) v[r] = *(const bf16x8*)(f + (((size_t)img * g.c_in + c0 + ch) * g.h + (yp - 1)) * g.w + x);
    }
    bf16 first = (bf16)0.f;                                // column xp0 - 1 of channel tid (threads 0 .. 63)
    if (tid < 64 && row_in && xp0 >= 1 && xp0 - 1 < g.w)
        first = f[(((size_t)img * g.c_in + c0 + tid) * g.h + (yp - 1)) * g.w + xp0 - 1];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = tid + r * 256, ch = i >> 3, q = i & 7;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int xl = 8 * q + e + 1;                  // padded column inside the tile
            if (xl < 64) tile[ch * PACKV_PITCH + xl] = v[r][e];
        }
    }
    if (tid < 64) tile[tid * PACKV_PITCH] = first;
    __syncthreads();
    const size_t prow = ((size_t)img * g.Hp + yp) * g.Wp;  // padded position of column 0 of this row
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = tid + r * 256;
        {   // position-major: 8 channels of one position
            const int xl = i >> 3, cq = i & 7;
            if (xp0 + xl < g.Wp) {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = tile[(cq * 8 + e) * PACKV_PITCH + xl];
                *(bf16x8*)(out + (prow + xp0 + xl) * g.c_in + c0 + cq * 8) = o;
            }
        }
        {   // channel-major: 8 positions of one channel
            const int ch = i >> 3, g8 = i & 7;
            if (outT && xp0 + 8 * g8 < g.Wp)
                *(bf16x8*)(outT + xt_index(c0 + ch, guard + (int)prow + xp0 + 8 * g8, PPT / 8)) =
                    *(const bf16x8*)(tile + ch * PACKV_PITCH + 8 * g8);
        }
    }
}

// weight with which frame index X (0 .. 8*len-1) contributes to cell `cell` of a line of `len`
// cells: the tent (1, 3, .. 15, 15, .. 3, 1)/16 around the cell, plus, for the first and last
// cell, the weight that edge replication folds back onto them
__device__ __forceinline__ float tap_weight(int X, int cell, int len)
{
    const int t = X - 8 * cell + 4;   // 0 .. 15 inside the tent
    float wgt = 0.f;
    if (t >= 0 && t < 16) wgt = (t < 8 ? 2 * t + 1 : 31 - 2 * t) * 0.0625f;
    if (cell == 0 && X < 4) wgt = 1.f;
    if (cell == len - 1 && X >= 8 * len - 4) wgt = 1.f;
    return wgt;
}

// T[img][c][cy][cx] = sum over valid pixels p with label c of wy(p, cy) * wx(p, cx).
// One block (256 threads) per cell row and run of 32 cells.  First every pixel column that can
// reach those cells (256 + 2 x 4 columns) adds its 16 rows' y-weights into a per-column table in
// LDS (the class index is data, so the table cannot live in registers); then one thread per
// (class, cell) applies the x-weights of the 16 columns under the cell.  All terms are
// multiples of 1/256 and the sums stay below 2^8 -- below 2^16 with 8-bit pixel weights -- so the
// result is exact in float32 and does not depend on the order of additions.
// colsum: CP x (LABEL_NCOL + 1) floats of LDS, CP >= number of classes; cnt_part: 4 words.
constexpr int LABEL_TX = 32;                 // 8-pixel column groups per block of this role
constexpr int LABEL_NCOL = LABEL_TX * 8 + 8;
__device__ __forceinline__ void label_adjoint_block(const int32_t* __restrict__ labels,
                                                    const uint8_t* __restrict__ wmap, float* __restrict__ T,
                                                    unsigned int* __restrict__ count, const Geo& g,
                                                    int block, float* colsum, unsigned int* cnt_part, int CP,
                                                    uint8_t* __restrict__ lab8)
{
    constexpr int NCOL = LABEL_NCOL, PITCH = LABEL_NCOL + 1;
    const int tid = threadIdx.x;
    const int tiles_x = (g.w + LABEL_TX - 1) / LABEL_TX;
    const int tx = block % tiles_x, cy = (block / tiles_x) % g.h, img = block / (tiles_x * g.h);
    const int hw = g.h * g.w;
    const int32_t* lab = labels + (size_t)img * g.H * g.W;
    const uint8_t* wm = wmap ? wmap + (size_t)img * g.H * g.W : nullptr;
    const int X0 = tx * LABEL_TX * 8 - 4;                  // frame column of table column 0
    const int Yt = 8 * cy - 4;                             // frame row of tent position 0
    unsigned int cnt = 0;     // valid labels (their weights) of this block's own 8 x 256 pixels
    // A thread takes table column tid and, the first NCOL - 256 threads, column tid + 256 as
    // well.  The loads of both columns are issued before either is worked on: one trip to memory
    // for the block instead of two.
    static_assert(NCOL > 256 && NCOL <= 512, "one or two columns per thread");
    const bool second = tid < NCOL - 256;
    int ys[2][16];
    unsigned int ws[2][16];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k == 1 && !second) break;
        const int Xc = min(max(X0 + tid + 256 * k, 0), g.W - 1);
        // the 16 rows under the tent (clamped, so that no load depends on a branch of its own)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const size_t at = (size_t)min(max(Yt + r, 0), g.H - 1) * g.W + Xc;
            ys[k][r] = lab[at];
            ws[k][r] = wm ? wm[at] : 1u;
        }
    }
    // (the table is cleared while the labels are on their way)
    for (int i = tid; i < CP * PITCH; i += 256) colsum[i] = 0.f;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k == 1 && !second) break;
        const int col = tid + 256 * k;
        const int X = X0 + col;
        const bool xin = X >= 0 && X < g.W;
        const bool own_col = col >= 4 && col < NCOL - 4;
        // label maps are piecewise constant: rows with the same label are added up in a register
        // and reach the table once per run (all terms are multiples of 1/256, so any grouping of
        // the additions gives the same float32 sum)
        int run_y = -1;
        float run = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int Y = Yt + r, y = ys[k][r];
            const bool ok = xin && Y >= 0 && Y < g.H && y != g.ignore_index && y >= 0 && y < g.C;
            const int yy = ok ? y : -1;
            if (yy != run_y) {
                if (run_y >= 0) colsum[run_y * PITCH + col] += run;
                run_y = yy;
                run = 0.f;
            }
            if (ok) {
                run += (float)ws[k][r] * tap_weight(Y, cy, g.h);
                if (own_col && r >= 4 && r < 12) cnt += ws[k][r];
            }
            // the block's own 8 x 256 pixels as bytes for the loss kernel, which reads them in every
            // pass: the class, or 255 where the pixel does not count (a quarter of the bytes)
            if (lab8 && xin && own_col && r >= 4 && r < 12)
                lab8[(size_t)img * g.H * g.W + (size_t)Y * g.W + X] = ok ? (uint8_t)y : (uint8_t)255;
        }
        if (run_y >= 0) colsum[run_y * PITCH + col] += run;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
    if ((tid & 63) == 0) cnt_part[tid >> 6] = cnt;
    __syncthreads();
    if (tid == 0) *count = cnt_part[0] + cnt_part[1] + cnt_part[2] + cnt_part[3];
    for (int i = tid; i < g.C * LABEL_TX; i += 256) {
        const int lc = i % LABEL_TX, c = i / LABEL_TX;
        const int cx = tx * LABEL_TX + lc;
        if (cx >= g.w) continue;
        // (the tent's weights, for the first and last cell folded back by the edge replication: see tap_weight;
        //  columns off the frame hold zero sums)
        const bool first = cx == 0, last = cx == g.w - 1;
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const float tent = (t < 8 ? 2 * t + 1 : 31 - 2 * t) * 0.0625f;
            const float wgt = (t < 8 ? first : last) ? 1.f : tent;
            acc += wgt * colsum[c * PITCH + 8 * lc + t];   // table column 8 * lc + t: X = 8 * cx - 4 + t
        }
        T[((size_t)img * g.C + c) * hw + cy * g.w + cx] = acc;
    }
}

}  // namespace st
