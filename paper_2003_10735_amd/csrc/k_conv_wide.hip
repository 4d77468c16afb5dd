// 3x3 convolution (forward, and data-gradient as a forward with mirrored taps) on the matrix cores with a tile
// twice as wide as that of k_conv_mfma.hip: for grids that give a compute unit more than one block.
//
// What binds those grids in the small-tile kernel (128 positions x 64 channels per block, 8 wavefronts that each
// hold four 32 x 32 accumulator tiles) is not its K loop but what surrounds it: one block owns the compute unit, so
// the matrix cores idle while it fills its pipeline, exchanges its partial sums and stores (about 5 of 14 us per
// round), and its 0.25 weight kilobytes and one activation kilobyte per MFMA cost energy that the clock then lacks
// (a long launch of dense MFMAs runs at 1.3 - 1.7 GHz here).  Hence:
//   * a block is 256 threads = 4 wavefronts, 96 positions x 128 channels; two blocks share a compute unit (at most
//     256 registers and 80 KB of LDS each), so one block's K loop covers the other's prologue, exchange and stores;
//   * a wavefront holds 64 channels x 96 positions, so each activation fragment read from LDS feeds two MFMAs and each
//     weight fragment three; the four are 2 channel halves x 2 K groups.
// The sums are those of the small tiles, bit for bit: of a stage's four fragments of 16 channels a wavefront takes two,
// adds each to accumulators of its own (2 x 6 tiles, 192 registers), and the four partial sums of an element meet
// in the same order.  So a frame's activations and logits do not depend on which tile serves it.  (Two
// chains of twice the length instead of four cost accuracy, 1.44e-7 against 1.11e-7 of the products' 2-norm at 256 input
// channels and 1.28e-7 against 0.92e-7 at 192, and made ReLU masks and roundings to bfloat16 those of another sum.)
// Operands take the same routes as in k_conv_mfma.hip (weights in fragment order straight to registers, activations
// from memory into swizzled LDS slabs, three of which rotate), with the weights of three steps in a ring of fragment
// pairs and the next step's activation fragments read while this step's MFMAs run.
// Measured, us per launch, small tiles -> this kernel:
//   4 x 90 x 160 cells, 320 -> 256 104 -> 95, data gradient 256 -> 256 85 -> 72, layer 2 with classifier 85 -> 74;
//   135 x 240, 256 -> 128 30.5 -> 26.4, 128 -> 128 22.2 -> 17, its data gradient 22 -> 16.8.
// 128 positions per block need 256 accumulators a lane, so one block per compute unit: that loses the overlap.  (With the two
// chains of twice the length they fit, and 4 x 90 x 160 cells took 81, 62 and 63 us.)
#include <algorithm>

#include "st_conv.hpp"
#include "st_kernels.hpp"

namespace st {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int CW_P = 3;                    // blocks of 32 positions per block
constexpr int CW_BM = 32 * CW_P;
constexpr int CW_BN = 128;                 // channels per block
constexpr int CW_OLD = CW_BN + 8;          // pitch of the staged output tile
constexpr int CW_STEPS = 6;                // steps of a stage per wavefront: three taps x two fragments of 16 channels
constexpr int CW_RING = 3;                 // steps whose weights are in registers or on their way
#define CW_F __builtin_amdgcn_sched_barrier(0);

// dynamic LDS: the three slabs, later the exchanged sums (three sets of P accumulator tiles per channel half), then the
// output tile
constexpr size_t CW_LDS = std::max(std::max((size_t)3 * (CW_BM + 2) * 128, (size_t)2 * 3 * CW_P * 4096), (size_t)CW_BM * CW_OLD * 2);
static_assert(2 * CW_LDS <= 160 * 1024, "two blocks per compute unit");

// EPI as for k_conv3x3_mfma: 0 bias + ReLU, 1 ReLU mask of a data gradient, 2 as 0 with the classifier, 3 plain
// float32 sums to a dense tensor.
template <int EPI>
__global__ void __launch_bounds__(256, 2) k_conv3x3_wide(ConvArgs a)
{
    constexpr int P = CW_P, BM = CW_BM, BN = CW_BN, SLAB = (BM + 2) * 128, STEPS = CW_STEPS, RING = CW_RING, OLD = CW_OLD;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    // (the arguments, XCD-aware tile order, several heads: as in k_conv3x3_mfma)
    asm volatile("" ::"s"(a.tiles_per_xcd), "s"(a.m_tiles), "s"(a.n_tiles), "s"(a.by_n_tiles.m), "s"(a.by_grp_tiles.m), "s"(a.grp_tiles), "s"(a.grp_pp),
                 "s"(a.X), "s"(a.Wq), "s"(a.wq_stride), "s"(a.cin), "s"(a.Wp));
    const int tile = (blockIdx.x % 8) * a.tiles_per_xcd + blockIdx.x / 8;
    if ((int)(blockIdx.x / 8) >= a.tiles_per_xcd || tile >= a.m_tiles * a.n_tiles) return;
    const int mt = fast_quot(tile, a.by_n_tiles), nt = tile - mt * a.n_tiles;
    const int grp = fast_quot(mt, a.by_grp_tiles);
    const int m0 = grp * a.grp_pp + (mt - grp * a.grp_tiles) * BM, n0 = nt * BN;
    const int m_end = (grp + 1) * a.grp_pp;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kgrp = wave >> 1;
    const int l32 = lane & 31, lhi = lane >> 5;

    f32x16 acc[2][2][P];      // [fragment of the K group][channel block][position block]
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int j = 0; j < P; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[n >> 1][n & 1][j][r] = 0.f;

    const int c_chunks = a.cin / 64, n_stages = 3 * c_chunks, kfr = a.cin >> 4;

    // Activations: slab rows are positions m0 - 1 .. m0 + BM (shifted by the kernel row), 64 channels each, 16-byte
    // chunk c of row r at c ^ ((r >> 1) & 7).  A load of a wavefront fills eight rows; wavefront w takes the groups
    // w, w + 4, .. and wavefront 0 the two rows behind them.  (Rows behind the grid lie in the guard, whose
    // length counts on tiles of at most 256 positions.)
    static_assert(BM <= 256, "guard rows");
    const int lrow = lane >> 3, lpc = lane & 7;
    const int xo = ((8 * wave + lrow) * a.cin + ((lpc ^ ((4 * wave + (lrow >> 1)) & 7)) << 3)) * 2;
    const int xo_rest = ((BM + lrow) * a.cin + ((lpc ^ (lrow >> 1)) << 3)) * 2;
    const int x32 = 32 * a.cin * 2;
    const char* xsp = (const char*)(a.X + ((long long)m0 - 1 - a.Wp) * a.cin);
    const long long x_row = ((long long)a.Wp * a.cin - (c_chunks - 1) * 64) * 2;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    int rd[3];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) rd[kw] = (l32 + kw) * 128 + (((kgrp * 4 + lhi) ^ (((l32 + kw) >> 1) & 7)) << 4);

    // Weights.  Slot n of K group k is channel block n ^ k of the wavefront's half, so that after the K loop every
    // wavefront keeps its slot 0 and hands slot 1 to the wavefront of the other K group.  (Channel blocks behind the
    // last one read zeros or another block's weights; their sums are dropped.)
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.Wq + grp * a.wq_stride), 0, (int)(a.wq_stride * 2), 0x00020000);
    unsigned wv[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) wv[n] = (unsigned)((((n0 >> 5) + 2 * wn + (n ^ kgrp)) * 9 * kfr + kgrp * 2) * 1024 + lane * 16);
    int w_soff = 0;
    const int w_row = (2 * kfr + 4) * 1024;
    int w_cc = 0, x_cc = 0;

    u32x4 wr[RING][2];        // weight fragments of step t in slot t % RING, refilled for the step RING ahead once used
    bf16x8 xb[P];             // activation fragments of the step in work, each replaced by the next step's once used

    // step t: tap column t / 2, channel fragment t % 2
    auto load_w = [&](int soff, int t) __attribute__((always_inline)) {
        const int s = soff + ((t >> 1) * kfr + (t & 1)) * 1024;
#pragma unroll
        for (int n = 0; n < 2; ++n) wr[t % RING][n] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wv[n], s, 0);
    };
    // (assembly, and M0: see k_conv3x3_mfma)
    auto dma = [&](int slab, int i) __attribute__((always_inline)) {
        const char* src = xsp + (long long)i * x32;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(xo), "s"(src),
                     "s"(lds0 + slab * SLAB + (i * 4 + wave) * 1024) : "memory");
    };
    auto dma_rest = [&](int slab) __attribute__((always_inline)) {
        if (wave == 0 && lane < 16)
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(xo_rest), "s"(xsp),
                         "s"(lds0 + slab * SLAB + BM * 128) : "memory");
    };
    auto read_x = [&](int slab, int t, int j) __attribute__((always_inline)) {
        return *(const bf16x8*)(smem_raw + slab * SLAB + (rd[t >> 1] ^ ((t & 1) << 5)) + j * 4096);
    };
    auto x_next = [&]() __attribute__((always_inline)) { if (++x_cc == c_chunks) { x_cc = 0; xsp += x_row; } else xsp += 128; };
    auto w_next = [&]() __attribute__((always_inline)) { if (++w_cc == c_chunks) { w_cc = 0; w_soff += w_row; } else w_soff += 4096; };
    // s_waitcnt vmcnt(N) alone
#define CW_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | 0x0F70)

    // One stage out of slab B.  FX: the activations of the stage two ahead start their way into slab (B + 2) % 3,
    // which every wavefront has left behind the barrier of the stage before.  NEXT: another stage follows; its
    // slab is waited for in front of the last step (everything but the loads this stage has issued by then must
    // have landed), because that step already reads the next stage's first fragments.
    auto stage = [&](auto B_, auto FX_, auto NEXT_) __attribute__((always_inline)) {
        constexpr int B = decltype(B_)::value;
        constexpr bool FX = decltype(FX_)::value, NEXT = decltype(NEXT_)::value;
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (NEXT && t == STEPS - RING) w_next();
            const bool last = t == STEPS - 1;
            if (last && NEXT) {
                constexpr int issued = 2 * (STEPS - 1) + (FX ? P : 0);
                CW_VMCNT(issued);
                __syncthreads();
                CW_F
            }
#pragma unroll
            for (int j = 0; j < P; ++j) {
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    acc[t & 1][n][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wr[t % RING][n]), xb[j], acc[t & 1][n][j], 0, 0, 0);
                CW_F
                if (!last) xb[j] = read_x(B, t + 1, j);
                else if (NEXT) xb[j] = read_x((B + 1) % 3, 0, j);
                if (FX && !last) {
                    // the stage's P activation loads, spread over the steps in front of the barrier
                    constexpr int GAPS = (STEPS - 1) * P;
                    const int at = t * P + j;
                    if (at * P / GAPS != (at + 1) * P / GAPS) dma((B + 2) % 3, at * P / GAPS);
                    if (at == 0) dma_rest((B + 2) % 3);
                }
                CW_F
            }
            if (t < STEPS - RING) load_w(w_soff, t + RING);
            else if (NEXT) load_w(w_soff, t - (STEPS - RING));
            CW_F
        }
        if (FX) x_next();
    };
    typedef std::integral_constant<int, 0> I0; typedef std::integral_constant<int, 1> I1; typedef std::integral_constant<int, 2> I2;
    const std::true_type yes; const std::false_type no;

#pragma unroll
    for (int i = 0; i < P; ++i) dma(0, i);
    dma_rest(0);
    x_next();
#pragma unroll
    for (int t = 0; t < RING; ++t) load_w(0, t);
    CW_F
#pragma unroll
    for (int i = 0; i < P; ++i) dma(1, i);
    dma_rest(1);
    x_next();
    CW_VMCNT(2 * RING + P);
    __syncthreads();
    CW_F
#pragma unroll
    for (int j = 0; j < P; ++j) xb[j] = read_x(0, 0, j);
    CW_F
    // (the number of stages is a multiple of three; the last three are written out)
    for (int s = 0; s + 3 < n_stages; s += 3) {
        stage(I0{}, yes, yes);
        stage(I1{}, yes, yes);
        stage(I2{}, yes, yes);
    }
    stage(I0{}, yes, yes);
    stage(I1{}, no, yes);
    stage(I2{}, no, no);
#undef CW_VMCNT
#undef CW_F

    // ---- what the epilogue needs from memory, on its way while the partial sums are exchanged
    constexpr int CHUNKS = BM * (BN / 8) / 256;      // 16-byte chunks of the output tile per thread
    const int cw = wn * 64 + kgrp * 32;              // this wavefront's 32 channels inside the tile
    u32x4 mk[EPI == 1 ? CHUNKS : 1];
    if (EPI == 1) {
#pragma unroll
        for (int k = 0; k < CHUNKS; ++k) {
            const int q = tid + 256 * k, p = q / (BN / 8), c = n0 + q % (BN / 8) * 8;
            mk[k] = *(const u32x4*)(a.mask + (size_t)min(m0 + p, m_end - 1) * a.cout + min(c, a.cout - 8));
        }
    }
    f32x4 bias[EPI == 0 || EPI == 2 ? 4 : 1];
    unsigned inside = 0;      // bit j: position 32 j + l32 of the tile lies on the grid
    if (EPI == 0 || EPI == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            bias[k] = *(const f32x4*)(a.bias + grp * a.bias_stride + min(n0 + cw + k * 8 + lhi * 4, a.cout - 4));
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (conv_cell(a, m0 + j * 32 + l32, m_end).inside) inside |= 1u << j;
    }
    f32x16 sum[P];            // this wavefront's 32 channels
    __syncthreads();
    {
        // number q = 2 kgrp + f of an element's four partial sums, added in ascending order.  K group 0 hands the sum of
        // its two over (set 0), K group 1 each of its own (sets 1 and 2).
        float* red = (float*)smem_raw + (size_t)wn * 3 * P * 1024 + lane * 4;     // [wn][set][P][4 register groups][64 lanes][4]
        auto put = [&](int set, int j, const f32x16& v) __attribute__((always_inline)) {
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                *(f32x4*)(red + ((set * P + j) * 4 + rq) * 256) = f32x4{v[rq * 4], v[rq * 4 + 1], v[rq * 4 + 2], v[rq * 4 + 3]};
        };
        auto get = [&](int set, int j) __attribute__((always_inline)) {
            f32x16 v;
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const f32x4 u = *(const f32x4*)(red + ((set * P + j) * 4 + rq) * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[rq * 4 + e] = u[e];
            }
            return v;
        };
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (kgrp == 0) put(0, j, acc[0][1][j] + acc[1][1][j]);
            else { put(1, j, acc[0][1][j]); put(2, j, acc[1][1][j]); }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (kgrp == 0) sum[j] = acc[0][0][j] + acc[1][0][j] + get(1, j) + get(2, j);
            else sum[j] = get(0, j) + acc[0][0][j] + acc[1][0][j];
        }
        __syncthreads();
    }
    if (EPI == 3) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const ConvCell cell = conv_cell(a, m0 + j * 32 + l32, m_end);
            if (cell.inside) {
                float* dst = a.dense + ((size_t)cell.img * a.dense_c * a.h + (cell.y - 1)) * a.w + (cell.x - 1);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int ch = n0 + cw + (r >> 2) * 8 + lhi * 4 + (r & 3);
                    if (ch < a.dense_c) dst[(size_t)ch * a.h * a.w] = sum[j][r];
                }
            }
        }
        return;
    }

    // classifier fragments (A operand: rows = classes, k = the half of this tile's channels that this wavefront multiplies)
    u32x4 w3f[EPI == 2 ? 4 : 1];
    if (EPI == 2) {
        const bf16* w3row = a.W3q + grp * a.w3_stride + (size_t)min(l32, a.n_cls - 1) * a.cout + lhi * 8;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const u32x4 v = *(const u32x4*)(w3row + min(n0 + (wave & 1) * 64 + ks * 16, a.cout - 16));
            w3f[ks] = l32 < a.n_cls ? v : u32x4{0u, 0u, 0u, 0u};
        }
    }
    bf16* Os = (bf16*)smem_raw;      // [BM][OLD]
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = sum[j][rg * 4 + e];
                if (EPI != 1) v = inside & (1u << j) ? fmaxf(v + bias[rg][e], 0.f) : 0.f;
                o[e] = (bf16)v;
            }
            *(bf16x4*)(Os + (j * 32 + l32) * OLD + cw + rg * 8 + lhi * 4) = o;
        }
    }
    __syncthreads();
    if (EPI == 2) {
        // D[class][position], 32 positions and half of the tile's channels per wavefront and turn: one share of the logits
        // per 64 channels, as from the small tiles
#pragma unroll 1
        for (int u = wave; u < 2 * P; u += 4) {
            const int j = u >> 1, half = wave & 1;
            if (n0 + half * 64 >= a.cout) continue;
            f32x16 z;
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 xf = *(const bf16x8*)(Os + (j * 32 + l32) * OLD + half * 64 + ks * 16 + lhi * 8);
                z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w3f[ks]), xf, z, 0, 0, 0);
            }
            const int mp = m0 + j * 32 + l32;
            if (mp < m_end) {
                float* zrow = a.zpart + ((size_t)(2 * nt + half) * a.PP + mp) * a.zpitch + lhi * 4;
#pragma unroll
                for (int gq = 0; gq < 4; ++gq)
                    if (gq * 8 + lhi * 4 < a.zpitch)
                        *(f32x4*)(zrow + gq * 8) = f32x4{z[gq * 4], z[gq * 4 + 1], z[gq * 4 + 2], z[gq * 4 + 3]};
            }
        }
    }
    // position-major: 16 bytes = 8 channels of one position; a data gradient is masked on the way (the mask is zero
    // on the border of the grid)
    if (EPI == 1 || a.Y) {
#pragma unroll
        for (int k = 0; k < CHUNKS; ++k) {
            const int q = tid + 256 * k, p = q / (BN / 8), c = q % (BN / 8) * 8;
            bf16x8 o = *(const bf16x8*)(Os + p * OLD + c);
            if (EPI == 1) {
                const bf16x8 m = __builtin_bit_cast(bf16x8, mk[k]);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (float)m[e] > 0.f ? o[e] : (bf16)0.f;
                *(bf16x8*)(Os + p * OLD + c) = o;
            }
            if (a.Y && m0 + p < m_end && n0 + c < a.cout) store_through(a.Y + (size_t)m0 * a.cout + n0, (unsigned)(p * a.cout + c) * 2, __builtin_bit_cast(u32x4, o));
        }
        if (EPI == 1) __syncthreads();
    }
    if (a.YT) {
        // channel-major: 16 bytes = 8 consecutive positions of one channel, a wavefront two such groups of 32
        // channels, through the transposing LDS read: in a group of 16 lanes, lane r names (position r / 4,
        // channels 4 (r % 4) .. + 3) and lane i receives channel i of four consecutive positions
        for (int u = wave; u < 2 * P * (BN / 32); u += 4) {
            const int pg = u / (BN / 32) * 2 + lhi, c = u % (BN / 32) * 32;
            const bf16* row = Os + (pg * 8 + ((lane & 15) >> 2)) * OLD + c + (lane & 16) + 4 * (lane & 3);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)row);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(row + 4 * OLD));
            const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            if (m0 + pg * 8 < m_end && n0 + c < a.cout)
                store_through(a.YT + xt_index(n0 + c, a.guard + m0 + u / (BN / 32) * 16, a.PPT / 8), lhi * 512 + l32 * 16, __builtin_bit_cast(u32x4, v));
        }
    }
}

// Which tile a layer runs with.  A launch takes about (blocks on the busiest compute unit) x (time of a block) + a
// constant, the time of a block being linear in the input channels.  Fitted, in microseconds, to sweeps over 7 000 to 74 000
// positions, 64 to 320 input and 128 and 256 output channels.  Where the choice changes it names the faster kernel or one within
// 2 % (plain forward passes, all small / all wide tiles: 90 x 160 cells, 256 -> 128 -> 128 34.3 / 42.2 us, two of them 57.3 / 58.2, four
// 106.3 / 101.3; two of them with 64 -> 128 -> 128 43.2 / 40.8; 75 x 110, 256 -> 256 -> 256 58.0 / 51.6; 100 x 178, 256 -> 128 -> 128
// 54.5 / 48.0; 120 x 213 59.3 / 59.5).
ConvTile conv_tile(const Geo& g, int cin, int cout)
{
    struct Shape { ConvTile t; float block, per64, launch; };
    static const Shape shapes[2] = {{{128, 64}, 4.3f, 1.53f, 1.0f}, {{CW_BM, CW_BN}, 2.4f, 2.03f, 3.6f}};
    ConvTile best = shapes[0].t;
    float best_t = 0.f;
    for (const Shape& s : shapes) {
        const int blocks = g.heads() * cdiv(g.padded_positions() / g.heads(), s.t.bm) * cdiv(cout, s.t.bn);
        const float t = cdiv(blocks, 256) * (s.block + s.per64 * (cin / 64)) + s.launch;
        if (&s == shapes || t < best_t) { best = s.t; best_t = t; }
    }
    // Small tiles on a chip they do not fill: quarter and half tiles, as long as each finds a compute unit of its own.  A block fetches its
    // channels' weights whatever its positions, so its time falls less than its work, but what a stage multiplies, the exchange and
    // the epilogue go with the positions; a second round would cost more than that saves.  us a launch, layer 1 / layer 2 with the classifier,
    // and what 128 positions take: 16 x 24 cells, 64 -> 64 -> 64 (tiles of 32) 3.9 / 4.2, were 5.2 / 5.3; 30 x 53, 256 -> 128 -> 128 (32)
    // 6.6 / 5.1, were 9.5 / 6.6; 60 x 107, 64 -> 64 -> 64 (32) 4.2 / 4.6, were 5.7 / 5.8; 60 x 107, 256 -> 128 -> 128 (64) 8.6 / 6.0, were
    // 10.1 / 6.8.
    if (best.bn == 64)
        for (int bm : {32, 64})
            if (g.heads() * cdiv(g.padded_positions() / g.heads(), bm) * cdiv(cout, 64) <= 256) { best.bm = bm; break; }
    return best;
}

// (a: everything but the tiling)
void conv3x3_wide(Ctx& c, const char* name, ConvArgs a, int epi, int heads)
{
    a.grp_tiles = cdiv(a.grp_pp, CW_BM);
    a.m_tiles = heads * a.grp_tiles;
    a.n_tiles = cdiv(a.cout, CW_BN);
    a.by_n_tiles = fast_div(a.n_tiles); a.by_grp_tiles = fast_div(a.grp_tiles);
    a.tiles_per_xcd = cdiv(a.m_tiles * a.n_tiles, 8);
    const dim3 grid(a.tiles_per_xcd * 8);
    auto go = [&](auto kernel) {
        ensure_dynamic_lds((const void*)kernel, CW_LDS);
        ST_LAUNCH(c, name, kernel, grid, dim3(256), CW_LDS, a);
    };
    if (epi == 3) go(k_conv3x3_wide<3>);
    else if (epi == 1) go(k_conv3x3_wide<1>);
    else if (epi == 2) go(k_conv3x3_wide<2>);
    else go(k_conv3x3_wide<0>);
}

}  // namespace st
