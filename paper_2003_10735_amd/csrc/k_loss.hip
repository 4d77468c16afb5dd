// Fused x8 bilinear up-sampling + per-pixel softmax cross-entropy + its gradient with respect
// to the low-resolution logits + predicted class + confusion counts, in one pass over the
// labels.  The up-sampled logits (n x C x 8h x 8w) are never written to memory.
//
// Interpolation (pixel centres at half-integers, edge replication): for a destination index
// 8q + j the two source cells and the weight of the second are
//     j <  4:  cells q-1, q      weight (2j + 9) / 16
//     j >= 4:  cells q,   q+1    weight (2j - 7) / 16
// and lerp(a, b, t) is evaluated as fma(t, b - a, a), first along x, then along y, every
// operation rounded once in float32.  The predicted class is decided on exactly these values.
//
// What depends on the labels but not on the logits is computed once per call
// (label_adjoint_block, a role of the launch that opens a call): with U the up-sampling operator
// and Y the one-hot label map,
//     T = U^T Y                      (exact in float32: sums of multiples of 1/256)
// Then, with P the softmax of the up-sampled logits on the valid pixels,
//     d loss / d z = (U^T P - T) / N_valid
//     loss         = ( sum_valid logsumexp  -  <T, z> ) / N_valid        (U z is linear in z)
// so the per-step kernel needs no per-class label test at all: per pixel and class it does one
// fma (interpolate), max/compare (prediction), fma + exp, add, and two fmas (U^T along y).
//
// Work split: one 512-thread block per tile of 1 x LOSS_TX groups of 8 x 8 pixels, two threads
// per pixel column (four pixels each).  A tile touches 3 x (LOSS_TX + 2) low-resolution cells;
// its share of U^T P for those cells goes to a slot of its own, and the consumer adds the (at
// most six) slots that meet in a cell in a fixed order.  No floating-point atomics here:
// results do not change from run to run.
#include "st_kernels.hpp"
#include "st_mfma.hpp"

namespace st {

// fixed order, separately rounded: d = b - a;  r = fma(t, d, a)
__device__ __forceinline__ float lerp1(float a, float b, float t)
{
    const float d = __fsub_rn(b, a);
    return __builtin_fmaf(t, d, a);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, true));
}
// sum over the 64 lanes, in lane 63
__device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_add<0x111, 0xF>(v);      // from the lanes 1, 2, 4 and 8 below in rows of 16
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);      // lane 15 of the row below, into rows 1 and 3
    return dpp_add<0x143, 0xC>(v);   // lane 31, into rows 2 and 3
}

constexpr int LOSS_THREADS = 2 * 8 * LOSS_TX;   // two threads per pixel column of the tile

// How a block finds its tile: tiles of a frame, tiles in a row of them, tiles of the call and of an XCD; and sizes of the
// call that would take products to form: logits of a frame, floats of a share.  (Offsets inside the tensors of logits, T and
// labels stay below 2^32 elements: the call's checks.)
struct LossGrid { FastDiv per_frame, per_row; int n_tiles, per_xcd; unsigned chw; size_t share; };

// What bounds it: instruction issue.  A pixel and class take ten instructions (one fma, half a maximum, compare, select, fma,
// exponential, addition, two fmas), and with four wavefronts per SIMD the time of a launch is proportional to all that a thread
// executes.  Around the pixels:
//   * logits are staged class-fastest, cell by cell: a thread reads and writes four classes at a time (20 LDS reads of 16 bytes
//     where it took 76 of 4), and the chunks of consecutive cells lie in different banks (pitch: an odd number of chunks);
//   * the x-adjoint, a weighted sum of four lanes per class and cell row, has the matrix core transpose 4 x 4 lanes and classes
//     (four v_mfma_f32_4x4x1 against unit vectors: exact), after which a lane holds the four columns of one class and
//     sums them itself: 12 instructions for four values, where sums across lanes took 28 and the wait states between them;
//   * the parts that meet in a cell lie in planes indexed by that cell, with zeros where there is none, so that the closing sum is
//     unconditional;
//   * a block asks for everything it needs from memory in one trip, with the divisions of its index as products.
// Launch with gradient / without, before -> now: 90 x 160 cells, 19 classes 14.2 -> 12.7 / 10.4 -> 9.1 us, 135 x 240 30.8 -> 25.8 / 21.3 -> 16.4,
// 4 x 90 x 160, 21 classes 51.9 -> 46.2 / 38 -> 31, 16 x 16, 9 classes 6.7 -> 5.7 / 5.4 -> 4.5.  d loss / d z against float64, mean of
// 30 cases: 5.02e-8 -> 4.91e-8 (2-norm).
//
// (up to 24 padded classes the kernel is held to 128 registers, so that two blocks share a
//  compute unit: the phases of one then fill the barriers and memory waits of the other)
// CP: classes rounded up to a multiple of four (the layout of the logit shares and of the slots); CA: the number
// of classes itself, CP - 3 .. CP -- the per-pixel arithmetic runs over exactly these, so a padded class costs no
// instruction.
template <int CP, int CA, bool GRAD>
__global__ void __launch_bounds__(LOSS_THREADS, (CP <= 24 ? 4 : 2))
k_loss(ZSrc zs, const uint8_t* __restrict__ labels, const uint8_t* __restrict__ wmap, const float* __restrict__ T,
       uint8_t* __restrict__ pred, float* __restrict__ slots, float* __restrict__ loss_part,
       unsigned long long* __restrict__ conf, Geo g, LossGrid lg, CountSum count)
{
    static_assert(LOSS_TY == 1 && LOSS_TX == 32, "one row group of 32 column groups per tile: the two halves of a block split its 8 pixel rows");
    constexpr int CW = LOSS_CW, CH = LOSS_CH, CELLS = CH * CW, NT = LOSS_THREADS;
    constexpr int QC = CP / 4;                            // chunks of four classes
    constexpr int PITCH = QC % 2 ? CP : CP + 4;           // floats from cell to cell in LDS
    constexpr int PLANE = CW * PITCH;
    __shared__ __attribute__((aligned(16))) float zt[CH * PLANE];      // logits of the touched cells
    // what the column groups hand to the cells, [half][upper, lower cell row of the half][part][cell column][class]; the parts:
    // to the left cell (from columns 0 - 3 of its group), to the own cell from columns 0 - 3, from columns 4 - 7, to the right cell
    __shared__ __attribute__((aligned(16))) float contrib[GRAD ? 16 * PLANE : 4];
    __shared__ __attribute__((aligned(16))) unsigned int conf_l[32 * 32];          // label x prediction counts of this tile
    __shared__ float wsum[NT / 64];

    const int tid = threadIdx.x;
    // XCD-aware tile order: consecutive blocks go to different XCDs, each with an L2 of its own.
    // Every XCD gets a contiguous run of tiles (a band of rows), so the three tiles that stage the
    // same row of cells run on one XCD and two of them find the row in its L2.
    // (A block without a tile goes along with tile 0 as far as the loads: asked any earlier, the question
    //  costs every block a trip of its own for the arguments.)
    const bool has_tile = (int)(blockIdx.x >> 3) < lg.per_xcd && (int)((blockIdx.x & 7) * lg.per_xcd + (blockIdx.x >> 3)) < lg.n_tiles;
    const int bid = has_tile ? (blockIdx.x & 7) * lg.per_xcd + (blockIdx.x >> 3) : 0;
    const int img = fast_quot(bid, lg.per_frame), tile = bid - img * (int)lg.per_frame.d;
    const int qy = fast_quot(tile, lg.per_row), tile_x = tile - qy * (int)lg.per_row.d;   // qy: row group = cell row
    const int C = g.C, hw = g.h * g.w;
    const unsigned own = (unsigned)img * lg.chw + (unsigned)(qy * g.w);     // class 0 of this tile row in a planar tensor
    const int cx0 = tile_x * LOSS_TX - 1, cy0 = qy - 1;  // cell of local (0, 0)

    // ---- stage the touched cells (edge replication = clamped read), four classes of a cell per thread.  (The classes
    //      beyond the last are staged as they come; nothing reads them.)
    //      All global loads of the prologue are issued before anything waits for one of them.
    constexpr int NZQ = (CELLS * QC + NT - 1) / NT;
    f32x4 zr[NZQ][4], bq[NZQ];
    {
        // (beyond the classes: zeros, from behind the end of the descriptor)
        const __amdgpu_buffer_rsrc_t bias = __builtin_amdgcn_make_buffer_rsrc((void*)(zs.b3 + (unsigned)g.head_of(img) * (unsigned)zs.b3_stride), 0, C * 4, 0x00020000);
#pragma unroll
        for (int k = 0; k < NZQ; ++k) {
            const int i = min(tid + k * NT, CELLS * QC - 1);
            const int cell = i / QC, chunk = i - cell * QC;
            const int r = cell / CW, lc = cell - r * CW;
            const int cx = min(max(cx0 + lc, 0), g.w - 1), cy = min(max(cy0 + r, 0), g.h - 1);
            const int mp = (img * g.Hp + cy + 1) * g.Wp + cx + 1;
            // up to four shares (one per 64 channels, float32 path 32); within a group of two an absent
            // share re-reads the last one (it is then not added), so that the loads of a group are
            // issued together.  Only loaded here: the sums wait until every load of the prologue
            // is on its way.
            const float* zp = zs.parts + ((unsigned)mp * CP + chunk * 4);
            zr[k][0] = *(const f32x4*)zp;
            zr[k][1] = *(const f32x4*)(zp + (zs.n_parts > 1 ? lg.share : 0));
            if (zs.n_parts > 2) {
                zr[k][2] = *(const f32x4*)(zp + 2 * lg.share);
                zr[k][3] = *(const f32x4*)(zp + (zs.n_parts > 3 ? 3 : 2) * lg.share);
            }
            bq[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(bias, chunk * 16, 0, 0));
        }
    }
    // T over the cells this tile owns, for the  - <T, z>  part of the loss (see the header): class i / 32, column i % 32.
    // (Classes that do not exist lie behind the end of the descriptor; columns are dropped below.)
    constexpr int NTT = (LOSS_TX * CP + NT - 1) / NT;
    float tv[NTT];
    const bool want_tz = T && loss_part;
    if (want_tz) {
        const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc((void*)(T + own), 0, (int)((lg.chw - (unsigned)(qy * g.w)) * 4u), 0x00020000);
#pragma unroll
        for (int k = 0; k < NTT; ++k) {
            const unsigned i = tid + k * NT, at = (i >> 5) * (unsigned)hw + tile_x * LOSS_TX + (i & 31);
            tv[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(trs, (int)(at * 4u), 0, 0));
        }
    }

    // Two threads per pixel column: `half` 0 takes the upper four pixels of the 8 (they
    // interpolate between cell rows qy-1 and qy), half 1 the lower four (rows qy and qy+1).
    const int half = __builtin_amdgcn_readfirstlane(tid >> 8), t = tid & (NT / 2 - 1);
    const int j = t & 7, tq = t >> 3;
    const int X = tile_x * LOSS_TX * 8 + t;
    const bool col_ok = X < g.W;
    const int Yb = qy * 8 + half * 4;    // first of this thread's four pixel rows
    // labels of this thread's 4 pixels, fetched before the barrier
    int lab4[4] = {255, 255, 255, 255};
    int wraw[4] = {1, 1, 1, 1};              // loss weight of each pixel
    if (labels) {
        const unsigned Xc = min(X, g.W - 1);
        const uint8_t* row = labels + (unsigned)((img * g.H + Yb) * g.W);
#pragma unroll
        for (int i = 0; i < 4; ++i) lab4[i] = (row + i * g.W)[Xc];
        if (wmap) {
            const uint8_t* wm = wmap + (unsigned)((img * g.H + Yb) * g.W);
#pragma unroll
            for (int i = 0; i < 4; ++i) wraw[i] = (wm + i * g.W)[Xc];
        }
    }
    // ---- every load of the prologue is issued
    if (!has_tile) {
        const int head = (int)blockIdx.x - ((lg.n_tiles + 7) & ~7);
        if (head < 0) return;
        // (a block behind the tiles: the pixel count of one head, a whole number)
        unsigned int* part = conf_l;
        unsigned long long total = 0;
        for (int i = tid; i < count.per_head; i += NT) total += count.counts[(size_t)head * count.per_head + i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) total += __shfl_down(total, off, 64);
        if ((tid & 63) == 0) { part[tid >> 6] = (unsigned int)total; part[16 + (tid >> 6)] = (unsigned int)(total >> 32); }
        __syncthreads();
        if (tid == 0) {
            total = 0;
            for (int w = 0; w < NT / 64; ++w) total += part[w] | ((unsigned long long)part[16 + w] << 32);
            count.n_valid[head] = total;
        }
        return;
    }
    // while they are on their way: what is cleared
    *(uint2*)(conf_l + 2 * tid) = make_uint2(0u, 0u);
    static_assert(2 * NT == 32 * 32, "two counters per thread");
    if (GRAD) {
        constexpr int QP = PITCH / 4;
        for (int i = tid; i < 32 * QP; i += NT) {
            const int pc = i / QP, part = (pc >> 1) & 3, which = pc & 1;
            const int cell = part == 0 ? 32 + which : part == 3 ? which : 33 * which;
            *(f32x4*)(contrib + (pc >> 1) * PLANE + cell * PITCH + (i - pc * QP) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // ---- from here on the loaded values are used
#pragma unroll
    for (int k = 0; k < NZQ; ++k) {
        const int i = tid + k * NT;
        const int cell = i / QC, chunk = i - cell * QC;
        // the shares in ascending order (each addition rounded on its own), then the bias
        f32x4 acc = zr[k][0];
        if (zs.n_parts > 1) acc += zr[k][1];
        if (zs.n_parts > 2) {
            acc += zr[k][2];
            if (zs.n_parts > 3) acc += zr[k][3];
            // (more than 256 channels in the second layer, float32 path 128)
            for (int s = 4; s < zs.n_parts; ++s) {
                const int ii = min(i, CELLS * QC - 1), cl = ii / QC, ch = ii - cl * QC;
                const int cx = min(max(cx0 + cl % CW, 0), g.w - 1), cy = min(max(cy0 + cl / CW, 0), g.h - 1);
                const int mp = (img * g.Hp + cy + 1) * g.Wp + cx + 1;
                acc += *(const f32x4*)(zs.parts + s * lg.share + ((unsigned)mp * CP + ch * 4));
            }
        }
        if (i < CELLS * QC) *(f32x4*)(zt + cell * PITCH + chunk * 4) = acc + bq[k];
    }
    __syncthreads();
    // the logits of this tile's own cells, as used below, for whoever wants the planar tensor; their product with T
    float loss_acc = 0.f;
    if (zs.z_out || want_tz) {
        float* zrow = zs.z_out ? zs.z_out + own : nullptr;
#pragma unroll
        for (int k = 0; k < NTT; ++k) {
            const unsigned i = tid + k * NT, lc = i & 31, c = i >> 5;
            const int cx = tile_x * LOSS_TX + lc;
            if ((int)c < C && cx < g.w) {
                const float z = zt[(CW + lc + 1) * PITCH + c];
                if (zrow) *(float*)((char*)zrow + (c * (unsigned)hw + cx) * 4u) = z;
                if (want_tz) loss_acc -= tv[k] * z;
            }
        }
    }

    // x-interpolated logits on this half's upper cell row and their difference to the lower one
    // (the y interpolation is fma(fy, difference, upper row): same roundings as lerp1)
    const float fx = (j < 4 ? 2 * j + 9 : 2 * j - 7) * 0.0625f;
    float Hu[CA], D[CA];
    {
        const float* zc = zt + (half * CW + tq + (j >> 2)) * PITCH;
#pragma unroll
        for (int q = 0; q < QC; ++q) {
            const f32x4 ul = *(const f32x4*)(zc + q * 4), ur = *(const f32x4*)(zc + PITCH + q * 4);
            const f32x4 ll = *(const f32x4*)(zc + PLANE + q * 4), lr = *(const f32x4*)(zc + PLANE + PITCH + q * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (q * 4 + e < CA) {
                    const float u = lerp1(ul[e], ur[e], fx);
                    Hu[q * 4 + e] = u;
                    D[q * 4 + e] = __fsub_rn(lerp1(ll[e], lr[e], fx), u);
                }
        }
    }
    float V[2][GRAD ? CA : 1];    // U^T along y: upper / lower cell row of the half
    if (GRAD) {
#pragma unroll
        for (int c = 0; c < CA; ++c) { V[0][c] = 0.f; V[1][c] = 0.f; }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // weight of the lower cell row: (9, 11, 13, 15) / 16 in the upper half, (1, 3, 5, 7) / 16 below
        const float fy = half ? (2 * i + 1) * 0.0625f : (2 * i + 9) * 0.0625f;
        float Z[CA];
#pragma unroll
        for (int c = 0; c < CA; ++c) Z[c] = __builtin_fmaf(fy, D[c], Hu[c]);
        // prediction: the largest logit, lowest index among equals
        float m = Z[0];
#pragma unroll
        for (int c = 1; c < CA; ++c) m = fmaxf(m, Z[c]);
        // (when nothing compares equal to the maximum -- NaN logits -- the answer is class 0)
        int best = 0;
#pragma unroll
        for (int c = CA - 1; c >= 0; --c) best = Z[c] == m ? c : best;
        if (pred && col_ok) (pred + (unsigned)((img * g.H + Yb + i) * g.W))[(unsigned)X] = (uint8_t)best;
        if (labels) {
            const float mb = -m * 1.44269504088896341f;
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < CA; ++c) {
                Z[c] = __builtin_amdgcn_exp2f(__builtin_fmaf(Z[c], 1.44269504088896341f, mb));
                sum += Z[c];
            }
            if (col_ok && lab4[i] < C) {     // (255: ignored or no class index)
                const float w = (float)wraw[i];
                loss_acc += w * __builtin_fmaf(__builtin_amdgcn_logf(sum), 0.693147180559945309f, m);
                atomicAdd(&conf_l[lab4[i] * 32 + best], 1u);
                if (GRAD) {
                    const float rs = w * __builtin_amdgcn_rcpf(sum);
                    const float wa = (1.f - fy) * rs, wb = fy * rs;
#pragma unroll
                    for (int c = 0; c < CA; ++c) {
                        V[0][c] = __builtin_fmaf(wa, Z[c], V[0][c]);
                        V[1][c] = __builtin_fmaf(wb, Z[c], V[1][c]);
                    }
                }
            }
        }
    }
    if (GRAD) {
        // edge replication for the first / last row group: the cell row outside the grid is the
        // border row itself
        if (qy == 0 && half == 0) {
#pragma unroll
            for (int c = 0; c < CA; ++c) { V[1][c] += V[0][c]; V[0][c] = 0.f; }
        }
        if (qy == g.h - 1 && half == 1) {
#pragma unroll
            for (int c = 0; c < CA; ++c) { V[0][c] += V[1][c]; V[1][c] = 0.f; }
        }
        // Adjoint of the x interpolation, summed over a group's 8 columns: columns 0-3 feed the left and the own cell, columns 4-7 the
        // own and the right one.  Lane n of a quad (four columns of one group) takes class 4 q + n of all four:
        // v_mfma_f32_4x4x1_16b_f32 gives lane n, register m, the sum of A of lane m times B of lane n, so with A = class 4 q + k
        // and B = 1 in lane k, 0 in the others, for k = 0 .. 3, lane n collects its class, unchanged.  (A column
        // that is not finite in one class -- a valid pixel with logits that are not -- is that in all.)
        const int n = t & 3, s = (t >> 2) & 1, q0 = tile_x * LOSS_TX + tq;
        // (edge replication: at the first / last column group the cell outside the grid is the border cell itself, so its
        //  weight goes to the own cell)
        const bool edge = s ? q0 == g.w - 1 : q0 == 0;
        float unit[4], w_side[4], w_own[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            unit[m] = n == m ? 1.f : 0.f;
            w_side[m] = edge ? 0.f : (s ? 2 * m + 1 : 7 - 2 * m) * 0.0625f;
            w_own[m] = 1.f - w_side[m];
        }
        float* to_side = contrib + (half * 8 + (s ? 3 : 0)) * PLANE + (tq + 2 * s) * PITCH + n;
        float* to_own = contrib + (half * 8 + 1 + s) * PLANE + (tq + 1) * PITCH + n;
#pragma unroll
        for (int q = 0; q < QC; ++q)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (q * 4 + k < CA) v = __builtin_amdgcn_mfma_f32_4x4x1f32(V[r][q * 4 + k], unit[k], v, 0, 0, 0);
                float side = v[0] * w_side[0], own = v[0] * w_own[0];
#pragma unroll
                for (int m = 1; m < 4; ++m) { side = __builtin_fmaf(v[m], w_side[m], side); own = __builtin_fmaf(v[m], w_own[m], own); }
                to_side[r * 4 * PLANE + q * 4] = side;
                to_own[r * 4 * PLANE + q * 4] = own;
            }
    }

    // ---- loss of this tile: wave sums, then the waves in order
    loss_acc = wave_sum(loss_acc);
    if ((tid & 63) == 63) wsum[tid >> 6] = loss_acc;
    __syncthreads();
    if (tid == 0 && loss_part) {
        float acc = wsum[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) acc += wsum[w];
        loss_part[bid] = acc;
    }
    if (conf && labels)
        for (int i = tid; i < C * 32; i += NT)
            if (conf_l[i]) atomicAdd(&conf[(unsigned)(img * C * C + (i >> 5) * C + (i & 31))], (unsigned long long)conf_l[i]);

    if (GRAD) {
        // Cell totals, four classes per thread: cell row 0 comes from the upper half, row 2 from the lower half, row 1 from both
        // (upper half first).  Cells outside the grid received nothing (their weight went to the border cells above).
        float* slot = slots + (size_t)bid * CP * CELLS;
#pragma unroll
        for (int k = 0; k < NZQ; ++k) {
            const int i = tid + k * NT, chunk = i / CELLS, cell = i - chunk * CELLS;
            const int r = cell / CW, lc = cell - r * CW;
            if (i < CELLS * QC) {
                const float* a = contrib + (r == 0 ? 0 : r == 1 ? 4 : 12) * PLANE + lc * PITCH + chunk * 4;
                // (in pairs: as near to the sum as any order gets)
                auto parts = [&](const float* p) __attribute__((always_inline)) {
                    return (*(const f32x4*)p + *(const f32x4*)(p + 3 * PLANE)) + (*(const f32x4*)(p + PLANE) + *(const f32x4*)(p + 2 * PLANE));
                };
                f32x4 v = parts(a);
                if (r == 1) v += parts(a + 4 * PLANE);
                float* dst = slot + chunk * 4 * CELLS + cell;
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[e * CELLS] = v[e];
            }
        }
    }
}

static int padded_classes(int C) { return (C + 3) / 4 * 4; }

size_t loss_slot_floats(const Geo& g)
{
    const LossTiling lt = loss_tiling(g);
    return (size_t)g.n * lt.tiles() * padded_classes(g.C) * LOSS_CH * LOSS_CW;
}

int loss_blocks(const Geo& g) { return g.n * loss_tiling(g).tiles(); }

template <int CP, int CA>
static void loss_launch(Ctx& c, const Geo& g, const ZSrc& zs, const uint8_t* labels, const uint8_t* wmap,
                        const float* T, uint8_t* pred, float* slots, float* loss_part, unsigned long long* conf, bool grad, const CountSum* count)
{
    const LossTiling lt = loss_tiling(g);
    const int n_tiles = g.n * lt.tiles();
    const int blocks = (n_tiles + 7) / 8 * 8 + (count ? g.heads() : 0);      // whole rounds over the eight XCDs
    const LossGrid lg = {fast_div(lt.tiles()), fast_div(lt.tiles_x), n_tiles, (n_tiles + 7) / 8, (unsigned)(g.C * g.h * g.w), (size_t)g.padded_positions() * CP};
    const CountSum cs = count ? *count : CountSum{nullptr, 0, nullptr};
    if (grad) {
        ST_LAUNCH(c, "upsample_ce_grad", (k_loss<CP, CA, true>), dim3(blocks), dim3(LOSS_THREADS), 0, zs, labels, wmap, T, pred,
                  slots, loss_part, conf, g, lg, cs);
    } else {
        ST_LAUNCH(c, "upsample_ce", (k_loss<CP, CA, false>), dim3(blocks), dim3(LOSS_THREADS), 0, zs, labels, wmap, T, pred, slots,
                  loss_part, conf, g, lg, cs);
    }
}

#define ST_FOR_CP(CALL)                                                                       \
    switch (padded_classes(g.C)) {                                                            \
    case 4: CALL(4); break;                                                                   \
    case 8: CALL(8); break;                                                                   \
    case 12: CALL(12); break;                                                                 \
    case 16: CALL(16); break;                                                                 \
    case 20: CALL(20); break;                                                                 \
    case 24: CALL(24); break;                                                                 \
    case 28: CALL(28); break;                                                                 \
    case 32: CALL(32); break;                                                                 \
    default: c.status = ST_ERR_SHAPE; break;                                                  \
    }

void loss_pass(Ctx& c, const Geo& g, const ZSrc& zs, const uint8_t* labels, const uint8_t* wmap, const float* T,
               uint8_t* pred, float* slots, float* loss_part, unsigned long long* conf, bool grad, const CountSum* count)
{
#define ST_ARGS c, g, zs, labels, wmap, T, pred, slots, loss_part, conf, grad, count
#define ST_CALL(CP)                                                                           \
    switch (CP - g.C) {                                                                       \
    case 0: loss_launch<CP, CP>(ST_ARGS); break;                                              \
    case 1: loss_launch<CP, CP - 1>(ST_ARGS); break;                                          \
    case 2: loss_launch<CP, CP - 2>(ST_ARGS); break;                                          \
    default: loss_launch<CP, CP - 3>(ST_ARGS); break;                                         \
    }
    ST_FOR_CP(ST_CALL)
#undef ST_CALL
#undef ST_ARGS
}

}  // namespace st
