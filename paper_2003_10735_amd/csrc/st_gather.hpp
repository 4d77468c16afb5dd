// d loss / d z of low-resolution cells from what the loss kernel left behind: the per-tile slots of
// U^T softmax (added in a fixed order: tile rows first), minus U^T of the one-hot labels, over N_valid.
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
    const int f = mp / frame, img = f < g.n ? f : g.n - 1;
    const int rr = mp - img * frame, y = rr / g.Wp, x = rr - y * g.Wp;
    const bool inside = mp < m_end && y >= 1 && y <= g.h && x >= 1 && x <= g.w;
    const int cy = inside ? y - 1 : 0, cx = inside ? x - 1 : 0;
    at.cell = GatherCell{img, cy, cx, inside};
    // the tiles whose cell window contains (cy, cx): up to 3 tile rows x 2 tile columns
    const int ty_top = (cy + 1) / LOSS_TY, tx_top = (cx + 1) / LOSS_TX;
    const int ty_hi = ty_top < lt.tiles_y ? ty_top : lt.tiles_y - 1, tx_hi = tx_top < lt.tiles_x ? tx_top : lt.tiles_x - 1;
    // offset of class 0 and a 0/1 weight: tiles that do not exist or do not touch the
    // cell read slot element 0 with weight 0, so that every load is unconditional
    const unsigned tile_floats = (unsigned)CP * (LOSS_CH * LOSS_CW);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int ty = ty_hi - 2 + a, tx = tx_hi - 1 + b;
            const int r = cy - (ty * LOSS_TY - 1), lc = cx - (tx * LOSS_TX - 1);
            const bool ok = inside && ty >= 0 && tx >= 0 && r >= 0 && r < LOSS_CH && lc >= 0 && lc < LOSS_CW;
            // (a call has fewer tiles than cells, and those are fewer than 2^25)
            const unsigned tile = ok ? img * lt.tiles() + ty * lt.tiles_x + tx : 0, in_tile = ok ? r * LOSS_CW + lc : 0;
            at.off[a][b] = (size_t)tile * tile_floats + in_tile;
            at.wgt[a][b] = ok ? 1.f : 0.f;
        }
    return at;
}

// Classes cq + STEP k (k < K) of padded position mp (< m_end: of this head) into v; 0 outside the grid,
// classes beyond the last hold its value.  All loads are issued before the first sum.
template <int K, int STEP>
__device__ __forceinline__ GatherCell gather_g(const float* __restrict__ slots, const float* __restrict__ T, unsigned long long nv,
                                               int CP, const LossTiling& lt, const Geo& g, int mp, int m_end, int cq, float (&v)[K])
{
    const int hw = g.h * g.w;
    const GatherAt at = gather_at(CP, lt, g, mp, m_end);
    const float inv_n = (at.cell.inside && nv) ? 1.0f / (float)nv : 0.f;
    const int cstride = LOSS_CH * LOSS_CW;
    const size_t tbase = (size_t)at.cell.img * g.C * hw + at.cell.cy * g.w + at.cell.cx;
    float sv[K][6], tv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int c = min(cq + STEP * k, g.C - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) sv[k][a * 2 + b] = slots[at.off[a][b] + (size_t)c * cstride];
        tv[k] = T[tbase + (size_t)c * hw];
    }
    __builtin_amdgcn_sched_barrier(0);
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
