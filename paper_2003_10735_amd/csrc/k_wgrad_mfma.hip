// Weight gradient of a 3x3 convolution on the matrix cores:
//
//   dW[o][tap][i] = sum_mp dY[o][mp] * X[i][mp + (kh-1)*Wp + (kw-1)]          (tap = kh*3 + kw)
//   db[o]         = sum_mp dY[o][mp]
//
// Both operands are read from their channel-major copies (positions contiguous), so that a
// lane's 8 reduction elements are 16 contiguous bytes and need no transposition.  dY is zero on
// the border of the padded grid, so the sum may run over all padded positions.
//
// One wavefront accumulates a 32 (o) x 32 (i) x 9 (taps) block (144 accumulator registers).  A unit is eight
// columns of two grid rows, y (lanes 0 .. 31) and y + 1 (lanes 32 .. 63), 16 positions: one dY fragment and, per kernel row
// kh, the X fragment kh - 1 rows further down (the row pitch of the padded grid is a multiple of 8, so all of them are aligned runs
// of the blocked channel-major layout); the kw = 0 and kw = 2 products use the dY fragment shifted by one
// position, built in registers (v_alignbyte with the element that enters from the unit before or behind, which the same
// lane holds) instead of loading shifted windows.  9 MFMAs per 4 loads.  A bigger block would need fewer loads per MFMA but leaves
// too few blocks to fill the chip without multiplying the partial copies.
// Why two rows: the three X fragments of a unit then are four row pieces of 512 bytes, two of them read twice at the same time
// and the second time mostly out of the L1 cache.  With a unit of 16 columns of one row they were six different ones, and a unit and
// wavefront took 4 KB from L2, 45 bytes per cycle and compute unit.  Read requests to L2 (TCP_TCC_READ_REQ_sum, millions a launch),
// before / now: 4 x 90 x 160 cells, 320 -> 256 -> 256 17.9 / 14.3, 135 x 240, 256 -> 128 -> 128 3.30 / 2.75, 90 x 160 1.52 / 1.33; the launches
// 143.9 / 130.1, 29.8 / 29.1 and 17.6 / 16.3 us (median under the profiler, one card; at 90 x 160 cells a wavefront has 49 units, and the
// first operands' way and the reduction are half the launch).  From memory it fetches more than before, not less (90 x 160 33.8 / 37.2 MiB:
// the rows of a pair are in two places).  The element that enters a shifted fragment now lies in the same lane; cross-lane
// permutes fetched it from the other half of the wavefront.
//
// The four wavefronts of a block own the same output block and a quarter each of the block's
// position range; they are added through LDS in a fixed order, and the grid's position splits
// are added by the optimiser kernel, also in a fixed order: no floating-point atomics.  The
// bias gradient (sums of dY over the positions) comes from one extra MFMA against a fragment of
// ones in the blocks of the first input-channel tile.
#include <algorithm>
#include <vector>

#include "st_kernels.hpp"
#include "st_mfma.hpp"
#include "st_wgrad.hpp"

namespace st {

struct WgradArgs {
    const bf16* dYT;   // channel-major copies in the blocked layout of xt_index()
    const bf16* XT;
    float* dW;         // [splits][stride] : this layer's weight block, [o][9][cin]
    float* db;         // [splits][stride] : this layer's bias block
    size_t split_stride;
    int cin, cout;        // channels of the gradient itself; the operands' are padded to multiples of 32
    int PPT, guard, Wp;
    int units_per_wave;   // units per wavefront
    int n_units;          // units of one head's positions: pairs of rows x groups of eight columns
    int o_tiles, i_tiles, splits, items_per_xcd;
    FastDiv by_tiles, by_splits, by_o_tiles, by_row;      // (o_tiles * i_tiles; splits; o_tiles; Wp / 8)
    // Several heads: head k owns the positions from 8-position group k * head_groups8 on and
    // writes its partial copies head_out_stride floats after head k - 1.
    int heads, head_groups8;
    // Groups from a head's first to the end of the one row behind its last: a border row of the next frame, or guard columns, zeros
    // either way.  Nothing behind it is an operand: with an odd number of rows the last pair reaches two rows further with
    // its X fragments, and there zeros are read.  (dY being zero in that pair's lower row is not enough: the rows behind
    // are the next client's, and zero times an infinity or a NaN of that client's is a NaN.)
    int end_groups;
    size_t head_out_stride;
};

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// One launch serves both 3x3 layers: blocks [0, blocks1) work on the first argument set, the rest
// on the second.  Every block pays the same fixed cost (pipeline fill, the reduction through LDS,
// the partial-result store) whatever its share of positions, so one grid that covers the chip
// once, with the position splits of the two layers balanced against each other, is much cheaper
// than two grids that each cover it once.
__global__ void __launch_bounds__(256) k_wgrad3x3_mfma(WgradArgs a1, WgradArgs a2, int blocks1)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const bool second = (int)blockIdx.x >= blocks1;
    const WgradArgs& a = second ? a2 : a1;
    const int bid = second ? blockIdx.x - blocks1 : blockIdx.x;

    // (the wavefront number through readfirstlane: the compiler then keeps everything derived
    //  from it -- the unit range, the loop counter, the load offsets -- in scalar registers)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    // XCD-aware order: consecutive blocks go to different XCDs; give each XCD a contiguous run
    // of work items in split-major order, so that one XCD's L2 only ever sees about 1/8 of the
    // positions (all channels) instead of every position of a few channels
    const int tiles = a.o_tiles * a.i_tiles;
    const int item = (bid % 8) * a.items_per_xcd + bid / 8;     // blocks1 is a multiple of 8
    if (bid / 8 >= a.items_per_xcd || item >= tiles * a.splits * a.heads) return;
    const int hsplit = fast_quot(item, a.by_tiles), tile = item - hsplit * tiles;
    const int head = fast_quot(hsplit, a.by_splits), split = hsplit - head * a.splits;
    // output-channel tile fastest: the blocks that stream the same X rows (same split, same
    // input-channel tile) are neighbours in the order, run on one XCD and share them in its L2
    const int it = fast_quot(tile, a.by_o_tiles), ot = tile - it * a.o_tiles;
    const int o0 = ot * 32, i0 = it * 32;

    // acc[0..8]: the nine taps; acc[9]: row sums of dY (bias gradient), only in blocks with it == 0
    f32x16 acc[10];
#pragma unroll
    for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

    const int unit0 = (split * 4 + wave) * a.units_per_wave;
    const int unit1 = min(unit0 + a.units_per_wave, a.n_units);
    // blocked layout: one 8-position group of 32 channels is 256 elements; lane (l32, lhi) reads
    // channel l32 of column group t % RG of row 2 (t / RG) + lhi, so each half of a wavefront's load is contiguous.
    // The operands are read through buffer descriptors, for X one per kernel row: the base (the unit before this
    // wavefront's first) sits in scalar registers, the lane offset is fixed, and every load takes one
    // scalar offset, the same for all four -- no address arithmetic at all in the vector unit, which the
    // K loop has no issue slots to spare for.
    const int NG = a.PPT >> 3;
    const int g0 = (a.guard >> 3) + head * a.head_groups8;     // this head's first 8-position group
    const int row_groups = a.Wp >> 3;   // one grid row = this many 8-position groups
    const unsigned row_bytes = (unsigned)row_groups * 512u;
    const int pair0 = fast_quot(unit0, a.by_row);
    int col = unit0 - pair0 * row_groups;                      // column group of the next unit to load
    const int first = pair0 * 2 * row_groups + col, before = first - (col ? 1 : row_groups + 1);    // groups of unit0 and unit0 - 1
    // (a descriptor ends at end_groups.  No load whose value is used has a scalar offset behind that end.)
    auto operand = [&](const bf16* base, int block, int group) __attribute__((always_inline)) {
        const long long left = ((long long)a.end_groups - group) * 512;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (((ptrdiff_t)block * NG + g0 + group) << 8)), 0,
                                                 (int)(unsigned)(left < 0xFFFFFFFFll ? left : 0xFFFFFFFFll), 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t yrs = operand(a.dYT, o0 >> 5, before);
    const __amdgpu_buffer_rsrc_t xrs[3] = {operand(a.XT, i0 >> 5, before - row_groups), operand(a.XT, i0 >> 5, before),
                                           operand(a.XT, i0 >> 5, before + row_groups)};
    const unsigned lane_off = lhi * row_bytes + l32 * 16;
    unsigned soff = (unsigned)(first - before) * 512u;         // of the next unit to load
    const bool want_bias = it == 0;
    const bf16 one = (bf16)1.0f;
    const bf16x8 ones = {one, one, one, one, one, one, one, one};

    // Operand ring: the loads of unit u + DEPTH - 1 are issued before the MFMAs of unit u, so
    // that an L2 round trip is covered by matrix work of the same wavefront (there is only one
    // wavefront per SIMD: the accumulators take most of the register file).
#ifndef ST_WGRAD_DEPTH
#define ST_WGRAD_DEPTH 8
#endif
    constexpr int DEPTH = ST_WGRAD_DEPTH;
    u32x4 ry[DEPTH], rx[DEPTH][3];
#define WG_LOAD_Y(SLOT, OFF) ry[SLOT] = __builtin_amdgcn_raw_buffer_load_b128(yrs, lane_off, (int)(OFF), 0);
#define WG_LOAD_X(SLOT, KH) rx[SLOT][KH] = __builtin_amdgcn_raw_buffer_load_b128(xrs[KH], lane_off, (int)soff, 0);
    // to the next unit: the next group of columns, behind the last one of a pair of rows the first of the next pair
#define WG_NEXT_A soff += 512u; ++col;
#define WG_NEXT_B { const bool end_ = col == row_groups; soff += end_ ? row_bytes : 0u; col = end_ ? 0 : col; }
    // The three taps of a kernel row differ by one position.  Moving the reduction index instead
    // of the window,
    //     dW[o][kh][kw][i] = sum_p dY[o][p - (kw - 1)] * X[i][p + (kh - 1) * Wp],
    // the kw = 0 / kw = 2 products use the same X fragment as kw = 1 and a dY fragment moved by
    // one position, which is built once per unit (not once per kernel row) in registers:
    // v_alignbyte over the lane's four dwords plus the one element that enters from the
    // neighbouring 8-position group, which this lane holds as the unit before (its dword 3) or behind (its dword 0).
    // (At the ends of a row what enters is the element of the next pair's first or the last pair's last column: both are
    //  border columns, where dY is zero, like in the guard columns.)
    u32x4 ymb[2], ypb[2];                 // dY at p - 1 / p + 1 of the unit in work and of the next one
    // In three parts, so that no gap between two MFMAs has to take more than three instructions.  (And without a loop:
    // the compiler would move the MFMAs in front behind it.)
#define WG_SHIFTED_A(PREV, SLOT, BUF)                                                           \
    ymb[BUF][0] = __builtin_amdgcn_alignbyte(ry[SLOT][0], ry[PREV][3], 2);                      \
    ymb[BUF][1] = __builtin_amdgcn_alignbyte(ry[SLOT][1], ry[SLOT][0], 2);                      \
    ymb[BUF][2] = __builtin_amdgcn_alignbyte(ry[SLOT][2], ry[SLOT][1], 2);
#define WG_SHIFTED_B(SLOT, NEXT, BUF)                                                           \
    ymb[BUF][3] = __builtin_amdgcn_alignbyte(ry[SLOT][3], ry[SLOT][2], 2);                      \
    ypb[BUF][3] = __builtin_amdgcn_alignbyte(ry[NEXT][0], ry[SLOT][3], 2);
#define WG_SHIFTED_C(BUF) ypb[BUF][0] = ymb[BUF][1]; ypb[BUF][1] = ymb[BUF][2]; ypb[BUF][2] = ymb[BUF][3];
#define WG_MMA(T, Y, KH, SLOT)                                                                  \
    acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(rx[SLOT][KH]), as_bf16x8(Y), acc[T], 0, 0, 0);
#define WG_F __builtin_amdgcn_sched_barrier(0);
    // One unit in slot D of the ring.  There is one wavefront per SIMD, so whatever this wavefront
    // issues between two MFMAs is all that can overlap them, and a lone wavefront issues one instruction in
    // about 7.7 cycles: an MFMA (33) hides three others of any kind, waits and scalar ones included, and each further one
    // costs those 7.7.  So no gap between this unit's nine MFMAs takes more: the loads of unit + DEPTH - 1, the
    // shifted fragments of unit + 1 and the step to the next unit to load, in a pinned order.
#define WG_UNIT(D, BIAS, LOADS)                                                                 \
    {                                                                                           \
        const int L_ = ((D) + DEPTH - 1) % DEPTH, N1_ = ((D) + 1) % DEPTH, N2_ = ((D) + 2) % DEPTH, B_ = (D) & 1; \
        if (BIAS) acc[9] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, as_bf16x8(ry[D]), acc[9], 0, 0, 0); \
        WG_MMA(0, ypb[B_], 0, D) WG_F                                                           \
        if (LOADS) WG_LOAD_Y(L_, soff) WG_F                                                     \
        WG_MMA(1, ry[D], 0, D) WG_F                                                             \
        if (LOADS) WG_LOAD_X(L_, 0) WG_F                                                        \
        WG_MMA(2, ymb[B_], 0, D) WG_F                                                           \
        if (LOADS) WG_LOAD_X(L_, 1) WG_F                                                        \
        WG_MMA(3, ypb[B_], 1, D) WG_F                                                           \
        if (LOADS) WG_LOAD_X(L_, 2) WG_F                                                        \
        WG_MMA(4, ry[D], 1, D) WG_F                                                             \
        WG_SHIFTED_A(D, N1_, 1 - B_) WG_F                                                       \
        WG_MMA(5, ymb[B_], 1, D) WG_F                                                           \
        WG_SHIFTED_B(N1_, N2_, 1 - B_) WG_F                                                     \
        WG_MMA(6, ypb[B_], 2, D) WG_F                                                           \
        WG_SHIFTED_C(1 - B_) WG_F                                                               \
        WG_MMA(7, ry[D], 2, D) WG_F                                                             \
        if (LOADS) { WG_NEXT_A } WG_F                                                           \
        WG_MMA(8, ymb[B_], 2, D) WG_F                                                           \
        if (LOADS) WG_NEXT_B WG_F                                                               \
    }
#define WG_LOOPS(BIAS)                                                                          \
    {                                                                                           \
        int u = unit0;                                                                          \
        for (; u + DEPTH <= unit1; u += DEPTH) {                                                \
            _Pragma("unroll") for (int d = 0; d < DEPTH; ++d) WG_UNIT(d, BIAS, true)            \
        }                                                                                       \
        /* fewer than DEPTH units are left and in the ring, but for dY of the unit behind the last */ \
        WG_LOAD_Y(DEPTH - 1, soff)                                                              \
        _Pragma("unroll") for (int d = 0; d < DEPTH - 1; ++d)                                   \
            if (u + d < unit1) WG_UNIT(d, BIAS, false)                                          \
    }

    static_assert(DEPTH % 2 == 0 && DEPTH >= 4, "two fragment buffers alternate; shifted fragments look two units ahead");
    if (unit0 < unit1) {
        // unit0 - 1 (guard columns make it readable) supplies the first left neighbours and
        // unit1 the last right neighbours
        // (all loads are unconditional: a load under a branch would force the compiler to wait for every outstanding load
        //  at the join; past the end of the range the slots hold what follows there, or zeros behind the head's end: no
        //  product takes them)
        WG_LOAD_Y(DEPTH - 1, 0)
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d) {
            WG_LOAD_Y(d, soff) WG_LOAD_X(d, 0) WG_LOAD_X(d, 1) WG_LOAD_X(d, 2)
            WG_NEXT_A WG_NEXT_B
        }
        WG_SHIFTED_A(DEPTH - 1, 0, 0) WG_SHIFTED_B(0, 1, 0) WG_SHIFTED_C(0)
        if (want_bias) WG_LOOPS(true) else WG_LOOPS(false)
    }
#undef WG_LOAD_Y
#undef WG_LOAD_X
#undef WG_NEXT_A
#undef WG_NEXT_B
#undef WG_SHIFTED_A
#undef WG_SHIFTED_B
#undef WG_SHIFTED_C
#undef WG_MMA
#undef WG_F
#undef WG_UNIT
#undef WG_LOOPS

    // ---- the wavefronts' blocks are added through LDS; every row of acc[9] holds the sums over the
    //      positions: row 0 lives in lanes 0 .. 31
    float* red = (float*)smem_raw;
    float* redb = red + 4 * 9 * 32 * 32;           // [4][32] sums of dY over the positions
    if (want_bias && lhi == 0) redb[wave * 32 + l32] = acc[9][0];
    wgrad_reduce_store<true>(acc, red, a.dW + head * a.head_out_stride + (size_t)split * a.split_stride, o0, i0, a.cout, a.cin);
    if (want_bias && tid < 32 && o0 + tid < a.cout) {
        float* db = a.db + head * a.head_out_stride + (size_t)split * a.split_stride;
        db[o0 + tid] = ((redb[tid] + redb[32 + tid]) + redb[64 + tid]) + redb[96 + tid];
    }
}

// Position splits of the two layers for the shared launch.  Every block pays a fixed cost (ring
// fill, the reduction through LDS, the partial-result store) on top of its units, blocks start in
// launch order on whichever compute unit is free, and every partial copy is read once more by the
// optimiser kernel.  The search simulates exactly that for every pair of split counts and keeps the
// shortest; among equals, fewer partial copies.
// bfloat16: units of 16 positions (9 MFMAs of 32 cycles), the fixed cost is about 22 of them.  (The kernel's units are pairs of rows: where
// a head has an odd number of them, half a row more than is counted here.)
// float32: units of 16 positions (54 MFMAs of 32 cycles); a launch takes some 10 us + 1.4 per unit, of which 4 units count as fixed (2: 120 x 200
// cells, 256 -> 128 -> 128, 0.7 % slower; 8, 14: within 0.3 % at nine sizes from 16 x 16 cells on).  By the float32 instruction: units of 8
// positions (36 MFMAs of 64 cycles).
void wgrad_splits_for(const Geo& g, WgradForm form, int* s1_out, int* s2_out)
{
    constexpr int n_cu = 256;
    const int fixed_units = form == WGRAD_BF16 ? 22 : form == WGRAD_F32 ? 4 : 3, reread_units_per_chip = form == WGRAD_BF16 ? 13 : 2;
    const int min_units = form == WGRAD_BF16 ? 8 : 2;       // units per wavefront where a layer is split at all
    const int tiles1 = g.heads() * cdiv(g.c1, 32) * cdiv(g.c_in, 32), tiles2 = g.heads() * cdiv(g.c2, 32) * cdiv(g.c1, 32);
    const int n_units = cdiv(g.padded_positions() / g.heads(), form == WGRAD_F32_FEW ? 8 : 16);
    int best1 = 1, best2 = 1;
    long best_cost = -1;
    // compute units with the same free time form a group: (time, how many)
    struct Group { long t; long n; };
    auto run = [](std::vector<Group>& gs, long blocks, long d) {
        long makespan = 0;
        while (blocks > 0) {
            size_t e = 0;
            for (size_t i = 1; i < gs.size(); ++i)
                if (gs[i].t < gs[e].t) e = i;
            const long k = std::min(gs[e].n, blocks), t = gs[e].t + d;
            gs[e].n -= k;
            if (gs[e].n == 0) gs.erase(gs.begin() + e);
            size_t j = 0;
            for (; j < gs.size(); ++j)
                if (gs[j].t == t) break;
            if (j < gs.size()) gs[j].n += k; else gs.push_back(Group{t, k});
            makespan = std::max(makespan, t);
            blocks -= k;
        }
        return makespan;
    };
    std::vector<Group> gs;
    for (int s1 = 1; s1 <= 16; ++s1) {
        if (s1 > 1 && cdiv(n_units, s1 * 4) < min_units) break;
        for (int s2 = 1; s2 <= 16; ++s2) {
            if (s2 > 1 && cdiv(n_units, s2 * 4) < min_units) break;
            const long d1 = cdiv(n_units, s1 * 4) + fixed_units, d2 = cdiv(n_units, s2 * 4) + fixed_units;
            const long n1 = (long)tiles1 * s1, n2 = (long)tiles2 * s2;
            // list scheduling on n_cu units, layer 1 first
            gs.assign(1, Group{0, n_cu});
            long makespan = run(gs, n1, d1);
            makespan = std::max(makespan, run(gs, n2, d2));
            const long cost = (makespan * n_cu + reread_units_per_chip * (n1 + n2)) * 64 + s1 + s2;
            if (best_cost < 0 || cost < best_cost) { best_cost = cost; best1 = s1; best2 = s2; }
        }
    }
    *s1_out = best1; *s2_out = best2;
}

static WgradArgs wgrad_args(const Plan& p, const bf16* dYT, const bf16* XT, float* dW, float* db, int cin,
                            int cout, int splits)
{
    WgradArgs a;
    a.dYT = dYT; a.XT = XT; a.dW = dW; a.db = db;
    a.split_stride = p.grad_stride;
    a.cin = cin; a.cout = cout; a.PPT = p.PPT; a.guard = p.guard; a.Wp = p.g.Wp;
    a.heads = p.g.heads();
    const int rows = p.g.n * p.g.Hp / a.heads;
    a.n_units = (rows + 1) / 2 * (p.g.Wp / 8);
    a.head_groups8 = p.g.Hp * p.g.Wp / 8;
    a.end_groups = (rows + 1) * (p.g.Wp / 8);
    a.head_out_stride = p.grad_stride * p.grad_copies;
    a.units_per_wave = cdiv(a.n_units, splits * 4);
    a.o_tiles = cdiv(cout, 32); a.i_tiles = cdiv(cin, 32);
    a.splits = splits;
    a.items_per_xcd = cdiv(a.o_tiles * a.i_tiles * splits * a.heads, 8);
    a.by_tiles = fast_div(a.o_tiles * a.i_tiles); a.by_splits = fast_div(splits); a.by_o_tiles = fast_div(a.o_tiles); a.by_row = fast_div(p.g.Wp / 8);
    return a;
}

// weight and bias gradients of layer 1 (dY = da1, X = features) and layer 2 (dY = da2, X = a1)
void wgrad3x3_mfma(Ctx& c, const Plan& p, const bf16* da1T, const bf16* featT, const bf16* da2T,
                   const bf16* a1T, float* grad)
{
    const Geo& g = p.g;
    const WgradArgs a1 = wgrad_args(p, da1T, featT, grad + p.po.W1, grad + p.po.b1, g.c_in, g.c1, p.splits1);
    const WgradArgs a2 = wgrad_args(p, da2T, a1T, grad + p.po.W2, grad + p.po.b2, g.c1, g.c2, p.splits2);
    const int blocks1 = a1.items_per_xcd * 8, blocks2 = a2.items_per_xcd * 8;
    const size_t smem = WGRAD_SMEM_BYTES;
    ensure_dynamic_lds((const void*)k_wgrad3x3_mfma, smem);
    ST_LAUNCH(c, "conv12_wgrad_mfma", k_wgrad3x3_mfma, dim3(blocks1 + blocks2), dim3(256), smem, a1, a2, blocks1);
}

}  // namespace st
