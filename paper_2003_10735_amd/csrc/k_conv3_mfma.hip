// The 1x1 classifier layer on the matrix cores (bfloat16 operands, float32 accumulation).
//
// Forward:   z[img][c][pos] = b3[c] + sum_o a2[pos][o] * W3[c][o]            (float32, planar)
// Backward:  da2[pos][o]    = [a2[pos][o] > 0] * sum_c g[c][pos] * W3[c][o]
//            dW3[c][o]      = sum_pos g[c][pos] * a2[pos][o]
//            db3[c]         = sum_pos g[c][pos]
// with g = d loss / d z rounded to bfloat16 where it enters a product.  The class dimension
// (<= 32) is padded to one 32-row MFMA tile with zeros.
#include <string.h>

#include "st_kernels.hpp"
#include "st_gather.hpp"
#include "st_mfma.hpp"
#include "st_finish.hpp"

namespace st {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ backward
// One block = C3B_BP consecutive padded positions (g is zero on the border).  The block first
// forms g = d loss / d z for its cells from what the loss kernel left behind -- the per-tile slots
// of U^T softmax (added in a fixed order: tile rows first), minus U^T of the one-hot labels, over
// N_valid -- rounds it to bfloat16 and stages it in LDS in both orientations.  W3 comes transposed
// and padded to 32 classes from the optimiser kernel ([channel][32]), so its MFMA A fragments are
// 16-byte loads straight from memory.
// Then
//   wavefront w < 4 computes da2 for positions 32 (w % 2) .. +31 and half of the channel tiles
//   (K = classes), and db3 for eight classes,
//   wavefront 4 + w computes dW3 for channel tiles w, w+4, ..  over all positions (K = positions),
// so no sum of theirs crosses wavefronts and the two products run side by side.  Partial dW3 / db3 go to one slot per block; the optimiser
// kernel adds the slots in order (only the rows of real classes are stored).  The block's a2
// tile is loaded once, position-major, before the first barrier (its latency overlaps the
// staging of g) and kept in LDS: the ReLU mask is read from it directly, the dW3 operand
// through the transposing LDS read.
// A block takes C2 channels of the layer: all of them, or (RUNS, heads with more than 256) the run of
// channels that blockIdx.y names, each run forming g for itself.
// The work per position is small and every phase is a chain of dependent memory round trips, so
// the block is kept small: the grid then covers the whole chip and each chain is short.  512 threads
// halve a thread's share of the gather and let the two products (and db3, once a serial loop over the
// positions in one wavefront) run side by side.  Against 256 threads that did one after the other, 8-step
// key frame at 90 x 160 cells, C2 = 128: 715 -> 704 us; with loop exits 797 -> 783; on larger grids, where
// other blocks fill the gaps, 0.1 to 0.6 % of a call.
constexpr int C3B_BP = 64, C3B_NT = 512;

// (one or two wavefronts per SIMD are all this kernel asks for: said explicitly, because the
//  compiler otherwise keeps to 128 registers and then issues the slot loads one at a time)
//
// FIN (early-exit form of the training call): the blocks behind the first `main_blocks` do the
// bookkeeping of the forward pass that came before (finish_block: loss, per-frame mean IoU, the
// metric for the host) instead -- it touches nothing this kernel reads or writes, and riding
// along saves that pass a launch of its own.
template <int C2, bool RUNS, bool FIN>
__global__ void __launch_bounds__(C3B_NT, 1)
k_conv3_bwd_mfma(const float* __restrict__ slots, const float* __restrict__ T,
                 const unsigned long long* __restrict__ n_valid, int CP, LossTiling lt,
                 const bf16* __restrict__ a2,
                 const bf16* __restrict__ W3T, bf16* __restrict__ da2, bf16* __restrict__ da2T,
                 float* __restrict__ part, Geo g, int PPT, int guard, int grp_blocks, FastDiv by_grp_blocks, int main_blocks, FinishArgs fin)
{
    // (what the first loads need, in one trip for the arguments)
    asm volatile("" ::"s"(slots), "s"(T), "s"(n_valid), "s"(CP), "s"(lt.tiles_x), "s"(lt.tiles_y), "s"(a2), "s"(W3T), "s"(g.n), "s"(g.h), "s"(g.w), "s"(g.Hp), "s"(g.Wp),
                 "s"(g.C), "s"(g.grouped), "s"(g.by_frame.d), "s"(g.by_frame.m), "s"(g.by_row.d), "s"(g.by_row.m));
    if (FIN && (int)blockIdx.x >= main_blocks) {
        if (!RUNS || blockIdx.y == 0) finish_block<true, C3B_NT>(fin, (int)blockIdx.x - main_blocks, 0);
        return;
    }
    constexpr int BP = C3B_BP, NT = C3B_NT;
    constexpr int OT = C2 / 32;            // channel tiles
    constexpr int OH = OT / 2;             // da2 channel tiles per wavefront
    constexpr int DW = (OT + 3) / 4;       // dW3 channel tiles per wavefront
    constexpr int KS = BP / 16;            // K steps of the dW3 product
    constexpr int GP = BP + 8;             // pitch of g_cp rows (positions)
    constexpr int GC = 32 + 8;             // pitch of g_pc rows (classes)
    constexpr int OLD = C2 + 8;            // pitch of the output tile
    static_assert(OT % 2 == 0, "two wavefronts share the channel tiles of a position half");
    __shared__ __attribute__((aligned(16))) bf16 g_cp[32 * GP];     // [class][position]
    __shared__ __attribute__((aligned(16))) bf16 g_pc[BP * GC];     // [position][class]
    __shared__ __attribute__((aligned(16))) bf16 Os[BP * OLD];      // da2 tile [position][channel]
    __shared__ __attribute__((aligned(16))) bf16 A2s[BP * OLD];     // a2 tile [position][channel]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave & 3;   // half: place among the four of its role
    const int l32 = lane & 31, lhi = lane >> 5;
    const int PP = g.padded_positions(), frame = g.Hp * g.Wp;
    // several heads: blocks are counted per frame (grp_blocks each), so that no block mixes the
    // positions -- and with them W3 and the partial sums -- of two heads
    // (tiles in bands per XCD: what the loss kernel and the layer-2 convolution left behind for a band of rows was written on the same XCD.
    //  Key frame at 90 x 160 cells 567.3 -> 563.4 us, 60 x 107 cells, 48 channels 212.5 -> 209.8, 4 x 90 x 160 7414 -> 7398)
    const int bid = xcd_band(blockIdx.x, main_blocks);
    const int head = g.grouped ? fast_quot(bid, by_grp_blocks) : 0;
    const int m0 = g.grouped ? head * frame + (bid - head * grp_blocks) * BP : bid * BP;
    const int m_end = g.grouped ? (head + 1) * frame : PP;
    const int k2 = RUNS ? g.k2 : C2, ch0 = RUNS ? blockIdx.y * C2 : 0;     // channel pitch; first channel of this block
    W3T += ((size_t)head * k2 + ch0) * 32;

    // ---- early loads: the block's a2 tile (position-major, 16 bytes per load) on its way to LDS.
    //      Both uses take it from there: the ReLU mask of the da2 part, and the dW3 part, whose
    //      reduction runs over the positions and therefore wants 8 consecutive positions of one
    //      channel per lane -- the transposing LDS read hands out exactly that, so the layer-2
    //      convolution need not leave a channel-major copy of a2 behind.
    const int pm = (half & 1) * 32 + l32;          // position (inside the block) for the da2 part
    const int t0 = (half >> 1) * OH;               // first channel tile of the da2 part
    constexpr int A2_CHUNKS = BP * (C2 / 8) / NT;  // 16-byte chunks of the tile per thread
    u32x4 a2v[A2_CHUNKS];
#pragma unroll
    for (int k = 0; k < A2_CHUNKS; ++k) {
        const int q = tid + NT * k, p = q / (C2 / 8), part8 = q - p * (C2 / 8);
        // (Rows past this head's last position repeat it, a border cell: zeros.  That d loss / d z is zero in those rows would not do:
        //  with several heads they are the next client's, and zero times an infinity of its activations is a NaN.)
        a2v[k] = *(const u32x4*)(a2 + (size_t)min(m0 + p, m_end - 1) * k2 + ch0 + part8 * 8);
    }
    // W3^T fragments of this wavefront's da2 tiles: rows = channels, k = 16 classes per step
    // (the dW3 wavefronts load them too: a load under a branch would be waited for at the join)
    bf16x8 wfr[OH][2];
#pragma unroll
    for (int t = 0; t < OH; ++t)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) wfr[t][ks] = *(const bf16x8*)(W3T + ((size_t)(t0 + t) * 32 + l32) * 32 + ks * 16 + lhi * 8);
    // ---- stage g (both orientations) and W3^T
    {
        const int p = tid & (BP - 1), cq = tid / BP;     // this thread: one position, every eighth class
        constexpr int NQ = NT / BP;
        float v[32 / NQ];
        gather_g<32 / NQ, NQ>(slots, T, n_valid + head, CP, lt, g, m0 + p, m_end, cq, v);
#pragma unroll
        for (int k = 0; k < 32 / NQ; ++k) {
            const int cc = cq + NQ * k;
            const bf16 q = (cc < g.C) ? (bf16)v[k] : (bf16)0.f;
            g_cp[cc * GP + p] = q;
            g_pc[p * GC + cc] = q;
        }
    }
#pragma unroll
    for (int k = 0; k < A2_CHUNKS; ++k) {
        const int q = tid + NT * k, p = q / (C2 / 8), part8 = q - p * (C2 / 8);
        *(u32x4*)(A2s + p * OLD + part8 * 8) = a2v[k];
    }
    __syncthreads();

    float* slot = part + (size_t)bid * (32 * k2 + 32);
    if (wave < 4) {
        // ReLU mask of this lane's position
        bf16x4 mk[OH][4];
#pragma unroll
        for (int t = 0; t < OH; ++t)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) mk[t][rg] = *(const bf16x4*)(A2s + pm * OLD + (t0 + t) * 32 + rg * 8 + lhi * 4);

        // ---- da2: D[o][pos] = sum_c W3T[o][c] * g[c][pos], two K steps cover 32 classes
        {
            f32x16 acc[OH];
#pragma unroll
            for (int t = 0; t < OH; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const bf16x8 gf = *(const bf16x8*)(g_pc + pm * GC + ks * 16 + lhi * 8);
#pragma unroll
                for (int t = 0; t < OH; ++t) {
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfr[t][ks], gf, acc[t], 0, 0, 0);
                }
            }
            // (a2 is zero on the border, and g is zero there too: border rows of da2 come out zero)
#pragma unroll
            for (int t = 0; t < OH; ++t)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    bf16x4 ov;
#pragma unroll
                    for (int e = 0; e < 4; ++e) ov[e] = (bf16)((float)mk[t][rg][e] > 0.f ? acc[t][rg * 4 + e] : 0.f);
                    *(bf16x4*)(Os + pm * OLD + (t0 + t) * 32 + rg * 8 + lhi * 4) = ov;
                }
        }
        // ---- db3: eight threads per class, eight positions each
        if (ch0 == 0) {
            const int c = tid >> 3, q = tid & 7;
            const bf16x8 gv = *(const bf16x8*)(g_cp + c * GP + q * 8);
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) s += (float)gv[e];
            s += __shfl_xor(s, 1, 64); s += __shfl_xor(s, 2, 64); s += __shfl_xor(s, 4, 64);
            if (q == 0 && c < g.C) slot[32 * k2 + c] = s;
        }
    } else {
        // ---- dW3: D[c][o] = sum_pos g[c][pos] * a2[pos][o] over this block's positions
#pragma unroll
        for (int d = 0; d < DW; ++d) {
            const int t = half + 4 * d;
            if (t < OT) {
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 gf = *(const bf16x8*)(g_cp + l32 * GP + ks * 16 + lhi * 8);
                    // B fragment: lane = channel l32 of tile t, positions 16 ks + 8 lhi .. + 7.  In a
                    // group of 16 lanes, lane r names the row (position r / 4, channels 4 (r % 4) .. + 3)
                    // and lane i receives channel i of positions 0 .. 3 of the group's rows: two reads.
                    const bf16* row = A2s + (ks * 16 + lhi * 8 + ((lane & 15) >> 2)) * OLD + t * 32 + (lane & 16) + 4 * (lane & 3);
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)row);
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(row + 4 * OLD));
                    const s16x8 xs = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gf, __builtin_bit_cast(bf16x8, xs), acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int c = (r >> 2) * 8 + lhi * 4 + (r & 3);
                    if (c < g.C) store_through(slot + ch0 + t * 32, (unsigned)(c * k2 + l32) * 4, acc[r]);    // (rows beyond the classes are never read)
                }
            }
        }
    }
    __syncthreads();

    // ---- write the da2 tile: position-major rows and channel-major 8-position groups
    for (int q = tid; q < BP * (C2 / 8); q += NT) {
        const int p = q / (C2 / 8), part8 = q % (C2 / 8);
        if (m0 + p < m_end)
            store_through(da2 + (size_t)m0 * k2 + ch0, (unsigned)(p * k2 + part8 * 8) * 2, *(const u32x4*)(Os + p * OLD + part8 * 8));
    }
    // (through the transposing LDS read, a wavefront two groups of 32 channels: lane r of 16 names position r / 4, channels 4 (r % 4) .. + 3, and
    //  lane i receives channel i of four consecutive positions)
#pragma unroll
    for (int u = wave; u < (BP / 16) * OT; u += NT / 64) {
        const int pg = u / OT * 2 + lhi, c = u % OT * 32;
        const bf16* row = Os + (pg * 8 + ((lane & 15) >> 2)) * OLD + c + (lane & 16) + 4 * (lane & 3);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)row);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(row + 4 * OLD));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        if (m0 + pg * 8 < m_end)
            store_through(da2T + xt_index(ch0 + c, guard + m0 + u / OT * 16, PPT / 8), lhi * 512 + l32 * 16, __builtin_bit_cast(u32x4, v));
    }
}

// blocks (and partial-sum slots) per head
int conv3_bwd_blocks(const Geo& g) { return cdiv(g.padded_positions() / g.heads(), C3B_BP); }
size_t conv3_bwd_slot_floats(const Geo& g) { return (size_t)32 * g.k2 + 32; }

void conv3_bwd_mfma(Ctx& c, const Plan& p, const float* slots, const float* T,
                    const unsigned long long* n_valid, const bf16* a2, const bf16* W3T,
                    bf16* da2, bf16* da2T, float* part, const FinishArgs* finish)
{
    const Geo& g = p.g;
    const int grp_blocks = conv3_bwd_blocks(g);
    const int main_blocks = g.heads() * grp_blocks;
    const int CP = (g.C + 3) / 4 * 4;   // class padding of the loss kernel's slots
    FinishArgs fin;
    memset(&fin, 0, sizeof(fin));
    if (finish) {
        if (g.grouped) { c.status = ST_ERR_ARG; return; }   // (the riding role serves one head)
        fin = *finish;
    }
    // with `finish`: one more block per frame and one for the loss
    const int run = g.k2 <= 256 ? g.k2 : g.k2 % 128 == 0 ? 128 : 64;     // channels per block
    const dim3 grid(main_blocks + (finish ? fin.fph + 1 : 0), g.k2 / run);
#define ST_C3B(C2, RUNS)                                                                                       \
    do {                                                                                                       \
        if (finish)                                                                                            \
            ST_LAUNCH(c, "conv3_bwd_mfma+finish_pass", (k_conv3_bwd_mfma<C2, RUNS, true>), grid, dim3(C3B_NT), 0, slots, T, \
                      n_valid, CP, p.lt, a2, W3T, da2, da2T, part, g, p.PPT, p.guard, grp_blocks, fast_div(grp_blocks), main_blocks, fin); \
        else                                                                                                   \
            ST_LAUNCH(c, "conv3_bwd_mfma", (k_conv3_bwd_mfma<C2, RUNS, false>), grid, dim3(C3B_NT), 0, slots, T, n_valid, CP, \
                      p.lt, a2, W3T, da2, da2T, part, g, p.PPT, p.guard, grp_blocks, fast_div(grp_blocks), main_blocks, fin);    \
    } while (0)
    if (run == g.k2) {
        switch (run) {
        case 64: ST_C3B(64, false); break;
        case 128: ST_C3B(128, false); break;
        case 192: ST_C3B(192, false); break;
        default: ST_C3B(256, false); break;
        }
    } else if (run == 128) ST_C3B(128, true);
    else ST_C3B(64, true);
#undef ST_C3B
}

}  // namespace st
