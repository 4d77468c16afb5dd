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

// The same for bfloat16 features with 16-byte reads (pack_vectors): one padded row yp (bz = img * Hp + yp), 64 channels (by)
// and 64 columns x0 .. x0 + 63 of the frame (bx) per block; column x is padded column x + 1.
//   channel-major: the eight padded columns 8 q .. 8 q + 7 are a thread's own chunk of eight columns moved by one, with the
//   last column of the chunk before it, which the lane before holds; no LDS.
//   position-major: the chunks go to LDS as they are, and the transposing read hands a lane eight channels of its column
//   (in a group of 16 lanes, lane r names (channel r / 4, columns 4 (r % 4) .. + 3) and lane i receives column i of four
//   channels).
// Bound by memory: at 135 x 240 cells, 256 channels, 17 MB are read and 34 MB written; alone it takes 12.9 us, 5 TB/s behind
// 3 us of launch.  (The chunks once went to LDS element by element, moved by one, and both copies came from there: the whole
// launch 22.7 us against 19.5.)
__device__ __forceinline__ void pack_features_vec_block(const bf16* __restrict__ f, bf16* __restrict__ out,
                                                        bf16* __restrict__ outT, const Geo& g, int PPT, int guard,
                                                        int bx, int by, int bz, bf16* tile)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const int x0 = bx * 64, c0 = by * 64;
    const int img = bz / g.Hp, yp = bz % g.Hp;
    const bool row_in = yp >= 1 && yp <= g.h;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bf16* row = f + ((size_t)img * g.c_in + c0) * g.h * g.w + (size_t)(yp - 1) * g.w;     // (read only if row_in)
    const size_t plane = (size_t)g.h * g.w;
    const int q = tid & 7, x = x0 + 8 * q;                 // a thread: columns x .. x + 7 of channels tid / 8 and tid / 8 + 32
    u32x4 v[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
    unsigned before[2] = {0u, 0u};                         // column x - 1 (upper half)
    if (row_in) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const bf16* src = row + ((tid >> 3) + 32 * r) * plane;
            if (x < g.w) v[r] = *(const u32x4*)(src + x);
            if (q == 0 && x0 > 0 && x0 - 1 < g.w) before[r] = (unsigned)__builtin_bit_cast(unsigned short, src[x0 - 1]) << 16;
        }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) *(u32x4*)(tile + ((tid >> 3) + 32 * r) * PACKV_PITCH + 8 * q) = v[r];
    const size_t prow = ((size_t)img * g.Hp + yp) * g.Wp;  // padded position of column 0 of this row
    if (outT) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const unsigned left = __builtin_amdgcn_update_dpp(0, (int)v[r][3], 0x111, 0xF, 0xF, true);     // lane - 1
            const unsigned prev = q ? left : before[r];
            const u32x4 o = {__builtin_amdgcn_alignbyte(v[r][0], prev, 2), __builtin_amdgcn_alignbyte(v[r][1], v[r][0], 2),
                             __builtin_amdgcn_alignbyte(v[r][2], v[r][1], 2), __builtin_amdgcn_alignbyte(v[r][3], v[r][2], 2)};
            if (x < g.Wp) *(u32x4*)(outT + xt_index(c0 + (tid >> 3) + 32 * r, guard + (int)prow + x, PPT / 8)) = o;
        }
    }
    __syncthreads();
    const int l16 = lane & 15, xl = 16 * wave + l16;       // this lane's column
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const int ch = hf * 32 + (lane >> 4) * 8;
        const bf16* at = tile + (ch + (l16 >> 2)) * PACKV_PITCH + 16 * wave + 4 * (l16 & 3);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)at);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(at + 4 * PACKV_PITCH));
        const s16x8 o = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        if (x0 + xl + 1 < g.Wp) *(s16x8*)(out + (prow + x0 + xl + 1) * g.c_in + c0 + ch) = o;
    }
    if (x0 == 0 && tid < 8) *(u32x4*)(out + prow * g.c_in + c0 + tid * 8) = u32x4{0u, 0u, 0u, 0u};     // padded column 0
}

// T[img][c][cy][cx] = sum over valid pixels p with label c of wy(p, cy) * wx(p, cx): the tent (1, 3, .. 15, 15, .. 3, 1)/16
// around the cell in either direction and, for the first and last cell, the weight that edge replication folds back
// onto them (1 on the outer half of the tent).
// One block (256 threads) per cell row and run of 31 cells, so that every pixel column that can reach those cells (248 + 2 x 4
// columns) has a thread.  A thread adds its column's 16 rows of y-weights into a per-column table in LDS (the class index is
// data, so the table cannot live in registers); then one thread per (class, cell) applies the x-weights of
// the 16 columns under the cell.  All terms are multiples of 1/256 and the sums stay below 2^8 -- below 2^16 with
// 8-bit pixel weights -- so the result is exact in float32 and does not depend on the order of additions.
// Bound by its chain of steps: 450 to 540 such blocks at 90 x 160 cells are all resident at once, and the launch ends
// when the slowest wavefront has walked its rows.  With 32 cells a block has 264 columns, the first wavefront walked two of
// them one after the other, and every run of rows was a read, an addition and a write of LDS in turn.  The launch with that
// role / with this one (and the packing role below): 60 x 107 cells, 96 channels 15.3 / 8.8 us, 90 x 160 cells, 256 channels
// 15.8 / 12.9 us, of which labels alone take 8.2, parameters 6.7 and packing 9.2.
// colsum: CP x LABEL_PITCH floats of LDS (16-byte aligned), CP >= number of classes; cnt_part: 4 words.
constexpr int LABEL_TX = 31;                 // 8-pixel column groups per block of this role
constexpr int LABEL_NCOL = LABEL_TX * 8 + 8;
constexpr int LABEL_PITCH = LABEL_NCOL + 4;  // (half-wavefronts that read two classes' rows use different banks)
static_assert(LABEL_NCOL == 256, "one column per thread");
__device__ __forceinline__ void label_adjoint_block(const int32_t* __restrict__ labels,
                                                    const uint8_t* __restrict__ wmap, float* __restrict__ T,
                                                    unsigned int* __restrict__ count, const Geo& g,
                                                    int block, float* colsum, unsigned int* cnt_part, int CP,
                                                    uint8_t* __restrict__ lab8)
{
    const int tid = threadIdx.x;
    const int tiles_x = (g.w + LABEL_TX - 1) / LABEL_TX;
    const int tx = block % tiles_x, cy = (block / tiles_x) % g.h, img = block / (tiles_x * g.h);
    const int hw = g.h * g.w;
    const int32_t* lab = labels + (size_t)img * g.H * g.W;
    const uint8_t* wm = wmap ? wmap + (size_t)img * g.H * g.W : nullptr;
    const int X = tx * LABEL_TX * 8 - 4 + tid;             // frame column of this thread
    const int Yt = 8 * cy - 4;                             // frame row of tent position 0
    // the 16 rows under the tent (clamped, so that no load depends on a branch of its own)
    int ys[16];
    unsigned int ws[16];
    {
        const int Xc = min(max(X, 0), g.W - 1);
#pragma unroll
        for (int r = 0; r < 16; ++r) ys[r] = lab[(size_t)min(max(Yt + r, 0), g.H - 1) * g.W + Xc];
#pragma unroll
        for (int r = 0; r < 16; ++r) ws[r] = 1u;
        if (wm) {
#pragma unroll
            for (int r = 0; r < 16; ++r) ws[r] = wm[(size_t)min(max(Yt + r, 0), g.H - 1) * g.W + Xc];
        }
    }
    // (the table is cleared while the labels are on their way)
    for (int i = tid; i < CP * LABEL_PITCH / 4; i += 256) ((float4*)colsum)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    unsigned int cnt = 0;     // valid labels (their weights) of this block's own 8 x 248 pixels
    {
        const bool xin = X >= 0 && X < g.W;
        const bool own_col = xin && tid >= 4 && tid < LABEL_NCOL - 4;
        const bool top = cy == 0, bottom = cy == g.h - 1;
        uint8_t* out8 = lab8 + (size_t)img * g.H * g.W + (size_t)(8 * cy) * g.W + X;
        // label maps are piecewise constant: rows with the same label are added up in a register
        // and reach the table once per run (all terms are multiples of 1/256, so any grouping of
        // the additions gives the same float32 sum; no other thread touches the column)
        int run_y = -1;
        float run = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // (rows above the frame: only in the tent's upper half of the first cell row, below it: the lower half of the last)
            const bool yin = (r >= 4 || !top) && (r < 12 || !bottom);
            const bool ok = xin && yin && ys[r] != g.ignore_index && (unsigned)ys[r] < (unsigned)g.C;
            const int yy = ok ? ys[r] : -1;
            if (yy != run_y) {
                if (run_y >= 0) unsafeAtomicAdd(&colsum[run_y * LABEL_PITCH + tid], run);
                run_y = yy;
                run = 0.f;
            }
            const float tent = (r < 8 ? 2 * r + 1 : 31 - 2 * r) * 0.0625f;
            const float wgt = (float)ws[r] * ((r < 8 ? top : bottom) ? 1.f : tent);
            run += ok ? wgt : 0.f;
            // the block's own 8 x 248 pixels as bytes for the loss kernel, which reads them in every
            // pass: the class, or 255 where the pixel does not count (a quarter of the bytes)
            if (r >= 4 && r < 12 && own_col) {
                cnt += ok ? ws[r] : 0u;
                out8[(size_t)(r - 4) * g.W] = ok ? (uint8_t)ys[r] : (uint8_t)255;
            }
        }
        if (run_y >= 0) unsafeAtomicAdd(&colsum[run_y * LABEL_PITCH + tid], run);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
    if ((tid & 63) == 0) cnt_part[tid >> 6] = cnt;
    __syncthreads();
    if (tid == 0) *count = cnt_part[0] + cnt_part[1] + cnt_part[2] + cnt_part[3];
    for (int i = tid; i < g.C * 32; i += 256) {
        const int lc = i & 31, c = i >> 5;
        const int cx = tx * LABEL_TX + lc;
        if (lc >= LABEL_TX || cx >= g.w) continue;
        // table column 8 * lc + t: X = 8 * cx - 4 + t (columns off the frame hold zero sums)
        const bool first = cx == 0, last = cx == g.w - 1;
        float acc = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4*)(colsum + c * LABEL_PITCH + 8 * lc + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = q * 4 + e;
                const float tent = (t < 8 ? 2 * t + 1 : 31 - 2 * t) * 0.0625f;
                acc += ((t < 8 ? first : last) ? 1.f : tent) * v[e];
            }
        }
        T[((size_t)img * g.C + c) * hw + cy * g.w + cx] = acc;
    }
}

}  // namespace st
