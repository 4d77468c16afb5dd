// d loss / d z of low-resolution cells from what the loss kernel left behind: the per-tile slots of
// U^T softmax, minus U^T of the one-hot labels, over N_valid.  The slots are added in a fixed order: tile row by tile row,
// in each the tile column with the cell before the one beside it, be that to the left or to the right.
#pragma once
#include "st_common.hpp"

namespace st {

struct GatherCell { int img, cy, cx; bool inside; };

// Where padded position mp lies (< m_end: of this head), and the floats of the slots that hold its share for
// class 0.  A call's slots may be more than 2^31 floats, so an offset is 64 bits wide.
struct GatherAt {
    GatherCell cell;
    size_t off[3][2];
    float wgt[3][2];
};

__host__ __device__ __forceinline__ GatherAt gather_at(int CP, const LossTiling& lt, const Geo& g, int mp, int m_end)
{
    GatherAt at;
    const int frame = g.Hp * g.Wp;
    const int f = fast_quot(mp, g.by_frame), img = f < g.n ? f : g.n - 1;
    const int rr = mp - img * frame, y = fast_quot(rr, g.by_row), x = rr - y * g.Wp;
    const bool inside = mp < m_end && y >= 1 && y <= g.h && x >= 1 && x <= g.w;
    const int cy = inside ? y - 1 : 0, cx = inside ? x - 1 : 0;
    at.cell = GatherCell{img, cy, cx, inside};
    // the tiles whose cell window contains (cy, cx): up to 3 tile rows, and beside the tile column with the cell the one next to
    // it if the cell is its first or last column.  From one tile row to the next a cell moves up by one row of the window, so the
    // offsets of a column are equally far apart.
    static_assert(LOSS_TY == 1, "a cell row is a tile row");
    const int tx = cx / LOSS_TX, in = cx % LOSS_TX;
    const int tx1 = in == 0 ? tx - 1 : tx + 1, in1 = in == 0 ? LOSS_TX : -1;
    const bool beside = (in == 0 || in == LOSS_TX - 1) && tx1 >= 0 && tx1 < lt.tiles_x;
    const unsigned tile_floats = (unsigned)CP * (LOSS_CH * LOSS_CW);
    // tile row cy, where the cell is row 1 of the window.  (A call has fewer tiles than cells, and those are fewer than 2^25.)
    const unsigned tile = (unsigned)(img * lt.tiles() + cy * lt.tiles_x + tx);
    const long long step = (long long)lt.tiles_x * tile_floats - LOSS_CW;
    const long long col[2] = {(long long)((size_t)tile * tile_floats) + (LOSS_CW + in + 1),
                              (long long)((size_t)(tile + tx1 - tx) * tile_floats) + (LOSS_CW + in1 + 1)};
    // a 0/1 weight: tiles that do not exist or do not touch the cell read slot element 0 with weight 0, so that every
    // load is unconditional.  (That element belongs to a cell outside the grid: zero, whatever the first frame holds.)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool ok = inside && (a > 0 || cy > 0) && (a < 2 || cy + 1 < lt.tiles_y) && (b == 0 || beside);
            at.off[a][b] = ok ? (size_t)(col[b] + (a - 1) * step) : 0;
            at.wgt[a][b] = ok ? 1.f : 0.f;
        }
    return at;
}

// Classes cq + STEP k (k < K) of padded position mp (< m_end: of this head) into v; 0 outside the grid,
// classes beyond the last hold its value.  cq: the same for all lanes.  All loads are issued before the first sum -- that of
// the pixel count among them, by a vector load: a scalar one would be waited for with the kernel's arguments.
template <int K, int STEP>
__device__ __forceinline__ GatherCell gather_g(const float* __restrict__ slots, const float* __restrict__ T, const unsigned long long* __restrict__ n_valid,
                                               int CP, const LossTiling& lt, const Geo& g, int mp, int m_end, int cq, float (&v)[K])
{
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 nv_raw = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
        __builtin_amdgcn_make_buffer_rsrc((void*)n_valid, 0, 8, 0x00020000), 0, 0, 0));
    cq = __builtin_amdgcn_readfirstlane(cq);
    const int hw = g.h * g.w;
    const GatherAt at = gather_at(CP, lt, g, mp, m_end);
    const int cstride = LOSS_CH * LOSS_CW;
    // (logits of a call are fewer than 2^30)
    const unsigned tbase = (unsigned)(at.cell.img * g.C * hw + at.cell.cy * g.w + at.cell.cx);
    float sv[K][6], tv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int c = min(cq + STEP * k, g.C - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) sv[k][a * 2 + b] = (slots + c * cstride)[at.off[a][b]];
        tv[k] = (T + (size_t)c * hw)[tbase];
    }
    __builtin_amdgcn_sched_barrier(0);
    unsigned nv_lo = nv_raw[0], nv_hi = nv_raw[1];
    asm volatile("" : "+v"(nv_lo), "+v"(nv_hi));      // (what is made of it stays behind the loads)
    const unsigned long long nv = nv_lo | (unsigned long long)nv_hi << 32;
    const float inv_n = (at.cell.inside && nv) ? 1.0f / (float)nv : 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float s = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) s = __builtin_fmaf(at.wgt[a][b], sv[k][a * 2 + b], s);
        v[k] = (s - tv[k]) * inv_n;
    }
    return at.cell;
}

}  // namespace st
