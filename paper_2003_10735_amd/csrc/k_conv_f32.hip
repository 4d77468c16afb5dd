// Float32 path: the head's contractions on the matrix cores at full float32 precision
// (v_mfma_f32_32x32x2_f32: float32 operands, float32 accumulation, each product and sum rounded once).
//
// One such instruction takes 64 cycles for 2048 multiply-adds and needs only 256 bytes of
// either operand, so these kernels are bound by the matrix cores as soon as every SIMD has work and
// the operands arrive in whole cache lines; LDS staging would buy nothing.  Hence:
//   * activations lie in runs of eight channels, [c / 8][position][8] (pos8_index): the B operand of a
//     tap -- 32 consecutive positions x 8 channels -- is one contiguous kilobyte at a constant offset,
//     and lane l holds channels 4 (l / 32) .. + 3 of position l % 32: the four pairs of k that four
//     MFMAs consume;
//   * weights lie in the matching fragment order (wfrag32_index), one contiguous kilobyte per
//     32 rows x 8 channels of a tap.
// So eight channels of one tap cost two coalesced 16-byte loads per lane and four MFMAs.
// Against a plain LDS-tiled GEMM on the vector units: 68 x 120 cells, 256 -> 128 -> 128, a 4-step call
// 4.62 -> 0.90 ms; 16 x 16 cells, 64 -> 64 -> 64, 1.52 -> 0.20 ms.
#include <algorithm>

#include "st_gather.hpp"
#include "st_kernels.hpp"
#include "st_mfma.hpp"
#include "st_wgrad.hpp"

namespace st {

// ------------------------------------------------------------------ 3x3 convolution
//   out[p][n] = epi( sum_{tap, c} X[p + shift(tap)][c] * W[n][tap][c] )        p: padded positions
// A block owns 32 positions x 32 output channels; its KG wavefronts split the reduction (taps x
// groups of eight channels) into contiguous runs and are added through LDS in ascending order.  Small
// tiles, because a frame has few of them: 68 x 120 cells and 128 channels make 1120, 4.4 per compute
// unit, where 64 x 64 tiles would make 280 and leave half the chip idle in the second round.  KG grows
// where there are few tiles (conv_f32), so that a 16 x 16 grid still reaches every compute unit.
struct Conv32Args {
    const float* X;       // pos8 layout, G groups of eight channels
    const float* Wf;      // fragment order, rows = output channels
    const float* bias;    // EPI 0, 2: zeros behind the last channel
    const float* mask;    // EPI 1: activation whose sign gates the gradient (layout of Y)
    float* Y;             // pos8 layout, GY groups (EPI 2: may be null)
    const float* W3f;     // EPI 2: [32 classes][w3_pitch], zero beyond the classes and channels
    float* zpart;         // EPI 2: this channel tile's share of the logits, [n-tile][padded position][zpitch]
    float* dense;         // EPI 3: [n][dense_c][h][w]
    int PP, Hp, Wp, h, w, G, GY, PPT, guard, w3_pitch, zpitch, dense_c;
    int m_tiles, n_tiles, tiles_per_xcd;
};

constexpr int C32_DEPTH = 4;    // operand sets on their way per wavefront: 3 x 256 cycles of MFMAs ahead

template <int EPI, int KG>
__global__ void __launch_bounds__(64 * KG) k_conv3x3_f32(Conv32Args a)
{
    extern __shared__ __attribute__((aligned(16))) float red[];    // [KG][4 register groups][64 lanes][4]
    // (consecutive blocks go to different XCDs: every XCD gets a contiguous run of position tiles)
    const int tile = (blockIdx.x % 8) * a.tiles_per_xcd + blockIdx.x / 8;
    if ((int)(blockIdx.x / 8) >= a.tiles_per_xcd || tile >= a.m_tiles * a.n_tiles) return;
    const int mt = tile / a.n_tiles, nt = tile % a.n_tiles;
    const int m0 = mt * 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    const int total = 9 * a.G, per = (total + KG - 1) / KG;
    const int i0 = wave * per, i1 = min(total, i0 + per);
    if (i0 < i1) {
        const float* wp = a.Wf + ((size_t)nt * total + i0) * 256;            // advances by 256 per item
        const float* xb = a.X + (size_t)(a.guard + m0) * 8;
        const unsigned wlane = lane * 4, xlane = l32 * 8 + lhi * 4;
        int tap = i0 / a.G, g = i0 - tap * a.G, li = i0;
        const float* xp = xb + ((ptrdiff_t)g * a.PPT + (tap / 3 - 1) * a.Wp + (tap % 3 - 1)) * 8;
        f32x4 ra[C32_DEPTH], rb[C32_DEPTH];
        // (past the end of the run the last item is loaded again and not used)
#define C32_LOAD(S)                                                                                \
        {                                                                                          \
            ra[S] = *(const f32x4*)(wp + wlane);                                                   \
            rb[S] = *(const f32x4*)(xp + xlane);                                                   \
            if (++li < i1) {                                                                       \
                wp += 256;                                                                         \
                if (++g == a.G) {                                                                  \
                    g = 0; ++tap;                                                                  \
                    xp = xb + (ptrdiff_t)((tap / 3 - 1) * a.Wp + (tap % 3 - 1)) * 8;               \
                } else xp += (ptrdiff_t)a.PPT * 8;                                                 \
            }                                                                                      \
        }
#define C32_MMA(S)                                                                                 \
        {                                                                                          \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                          \
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ra[S][e], rb[S][e], acc, 0, 0, 0);      \
        }
#pragma unroll
        for (int d = 0; d < C32_DEPTH; ++d) C32_LOAD(d)
        int i = i0;
        for (; i + C32_DEPTH <= i1; i += C32_DEPTH) {
#pragma unroll
            for (int d = 0; d < C32_DEPTH; ++d) { C32_MMA(d) C32_LOAD(d) }
        }
#pragma unroll
        for (int d = 0; d < C32_DEPTH - 1; ++d)
            if (i + d < i1) C32_MMA(d)
#undef C32_LOAD
#undef C32_MMA
    }
#pragma unroll
    for (int rq = 0; rq < 4; ++rq)
        *(f32x4*)(red + ((wave * 4 + rq) * 64 + lane) * 4) = f32x4{acc[rq * 4], acc[rq * 4 + 1], acc[rq * 4 + 2], acc[rq * 4 + 3]};
    __syncthreads();

    // wavefront rq < 4 finishes channels 8 rq .. + 7 of the tile: a lane holds 4 channels of one position
    const int rq = wave, ct = rq * 8 + lhi * 4, ch = nt * 32 + ct;
    const int frame = a.Hp * a.Wp;
    const int mp = m0 + l32;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (rq < 4) {
        const int img = mp / frame, rr = mp - img * frame, y = rr / a.Wp, x = rr - y * a.Wp;
        const bool inside = mp < a.PP && y >= 1 && y <= a.h && x >= 1 && x <= a.w;
#pragma unroll
        for (int k = 0; k < KG; ++k) v += *(const f32x4*)(red + ((k * 4 + rq) * 64 + lane) * 4);
        const size_t at = ((size_t)(nt * 4 + rq) * a.PPT + a.guard + mp) * 8 + lhi * 4;
        const bool stored = nt * 4 + rq < a.GY && mp < a.PP;
        if (EPI == 0 || EPI == 2) {
            const f32x4 b = *(const f32x4*)(a.bias + ch);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = inside ? fmaxf(v[e] + b[e], 0.f) : 0.f;
        } else if (EPI == 1) {
            f32x4 m = {0.f, 0.f, 0.f, 0.f};
            if (stored) m = *(const f32x4*)(a.mask + at);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = inside && m[e] > 0.f ? v[e] : 0.f;
        }
        if (EPI == 3) {
            if (inside) {
                float* dst = a.dense + (((size_t)img * a.dense_c + ch) * a.h + (y - 1)) * a.w + (x - 1);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ch + e < a.dense_c) dst[(size_t)e * a.h * a.w] = v[e];
            }
        } else if (stored && a.Y) *(f32x4*)(a.Y + at) = v;
    }
    if (EPI == 2) {
        // the classifier rides along: what this lane holds is the B operand of four MFMAs against
        // W3 (rows = classes, k = the 8 channels of this wavefront); the four wavefronts' sums
        // meet in LDS.  (All shares of the logits: one per 32 channels.)
        __syncthreads();       // the partial sums are read
        if (rq < 4) {
            f32x16 z;
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = 0.f;
            const f32x4 w3 = *(const f32x4*)(a.W3f + (size_t)l32 * a.w3_pitch + ch);
#pragma unroll
            for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_32x32x2f32(w3[e], v[e], z, 0, 0, 0);
            float* zr = red;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4*)(zr + ((rq * 4 + q) * 64 + lane) * 4) = f32x4{z[q * 4], z[q * 4 + 1], z[q * 4 + 2], z[q * 4 + 3]};
        }
        __syncthreads();
        if (rq < 4 && mp < a.PP && rq * 8 + lhi * 4 < a.zpitch) {     // (here rq: classes 8 rq .. + 7)
            const float* zr = red;
            f32x4 s = *(const f32x4*)(zr + (rq * 64 + lane) * 4);
#pragma unroll
            for (int k = 1; k < 4; ++k) s += *(const f32x4*)(zr + ((k * 4 + rq) * 64 + lane) * 4);
            *(f32x4*)(a.zpart + ((size_t)nt * a.PP + mp) * a.zpitch + rq * 8 + lhi * 4) = s;
        }
    }
}

template <int EPI, int KG>
static void conv_f32_launch(Ctx& c, const char* name, const Conv32Args& a, int blocks)
{
    const size_t smem = (size_t)KG * 1024 * sizeof(float);
    ensure_dynamic_lds((const void*)k_conv3x3_f32<EPI, KG>, smem);
    ST_LAUNCH(c, name, (k_conv3x3_f32<EPI, KG>), dim3(blocks), dim3(64 * KG), smem, a);
}

// cin, cout: channels of the layer as run here (exchanged for a data gradient)
static void conv_f32(Ctx& c, const char* name, const Plan& p, int epi, const float* X, const float* Wf, int cin, int cout,
                     const float* bias, const float* mask, float* Y, const float* W3f, float* zpart, float* dense)
{
    const Geo& g = p.g;
    Conv32Args a;
    a.X = X; a.Wf = Wf; a.bias = bias; a.mask = mask; a.Y = Y; a.W3f = W3f; a.zpart = zpart; a.dense = dense;
    a.PP = g.padded_positions(); a.Hp = g.Hp; a.Wp = g.Wp; a.h = g.h; a.w = g.w;
    a.G = cdiv(cin, 8); a.GY = cdiv(cout, 8); a.PPT = p.PPT; a.guard = p.guard;
    a.w3_pitch = cdiv(g.c2, 32) * 32; a.zpitch = (g.C + 3) / 4 * 4; a.dense_c = cout;
    a.m_tiles = cdiv(a.PP, 32); a.n_tiles = cdiv(cout, 32);
    const int tiles = a.m_tiles * a.n_tiles;
    a.tiles_per_xcd = cdiv(tiles, 8);
    const int blocks = a.tiles_per_xcd * 8;
    // as many wavefronts per tile as it takes to give each of the 1024 SIMDs two
    auto go = [&](auto e) {
        constexpr int E = decltype(e)::value;
        if (tiles >= 512) conv_f32_launch<E, 4>(c, name, a, blocks);
        else if (tiles >= 256) conv_f32_launch<E, 8>(c, name, a, blocks);
        else conv_f32_launch<E, 16>(c, name, a, blocks);
    };
    switch (epi) {
    case 0: go(std::integral_constant<int, 0>{}); break;
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    default: go(std::integral_constant<int, 3>{}); break;
    }
}

// ------------------------------------------------------------------ weight gradient
//   dW[o][tap][i] = sum_p dY[p][o] * X[p + shift(tap)][i],    db[o] = sum_p dY[p][o]
// One wavefront accumulates 32 (o) x 32 (i) x 9 (taps), k = positions.  The two values of k of an MFMA are
// not neighbours but the same place in the two halves of the wavefront's position range: a lane then
// walks its half one position at a time, and the three taps of a kernel row are the values it holds
// for the previous, this and the next position -- no shifting across lanes.  Per position four
// 4-byte loads (dY, and X in three rows) feed nine MFMAs (576 cycles).
// The rest (four wavefronts per block added through LDS, position splits added by the optimiser
// kernel, both layers in one launch) is as for the bfloat16 kernel.
struct Wgrad32Args {
    const float* dY; const float* X; float* dW; float* db;
    size_t split_stride;
    int cin, cout, GX, GY, PP, PPT, guard, Wp, len;       // len: positions per wavefront, even
    int o_tiles, i_tiles, splits, items_per_xcd;
};

__global__ void __launch_bounds__(256) k_wgrad3x3_f32(Wgrad32Args a1, Wgrad32Args a2, int blocks1)
{
    extern __shared__ __attribute__((aligned(16))) float red[];
    const bool second = (int)blockIdx.x >= blocks1;
    const Wgrad32Args& a = second ? a2 : a1;
    const int bid = second ? blockIdx.x - blocks1 : blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int tiles = a.o_tiles * a.i_tiles;
    const int item = (bid % 8) * a.items_per_xcd + bid / 8;
    if (bid / 8 >= a.items_per_xcd || item >= tiles * a.splits) return;
    const int split = item / tiles, tile = item - split * tiles;
    const int o0 = (tile % a.o_tiles) * 32, i0 = (tile / a.o_tiles) * 32;

    f32x16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    float bsum = 0.f;

    const int r0 = (split * 4 + wave) * a.len, r1 = min(r0 + a.len, a.PP);   // (PP is a multiple of eight)
    const int S = max(r1 - r0, 0) >> 1;
    if (S > 0) {
        // (channels beyond the last group re-read it: their sums are dropped at the end)
        const float* yb = a.dY + ((size_t)min((o0 + l32) >> 3, a.GY - 1) * a.PPT + a.guard + r0 + lhi * S) * 8 + (l32 & 7);
        const float* xb = a.X + ((size_t)min((i0 + l32) >> 3, a.GX - 1) * a.PPT + a.guard + r0 + lhi * S) * 8 + (l32 & 7);
        constexpr int D = 8;
        // slot s of the ring holds dY of position s (mod 8) and X of position s - 1.  Loads run up to seven
        // positions past the half (guard positions make them readable).
        float ry[D], rx[D][3];
#define W32_LOAD(S_, T)                                                                            \
        {                                                                                          \
            ry[S_] = yb[(T) * 8];                                                                  \
            _Pragma("unroll") for (int kh = 0; kh < 3; ++kh) rx[S_][kh] = xb[((T) - 1 + (kh - 1) * a.Wp) * 8]; \
        }
#define W32_MMA(S_)                                                                                \
        {                                                                                          \
            bsum += ry[S_];                                                                        \
            _Pragma("unroll") for (int kh = 0; kh < 3; ++kh)                                       \
            _Pragma("unroll") for (int kw = 0; kw < 3; ++kw)                                       \
                acc[kh * 3 + kw] = __builtin_amdgcn_mfma_f32_32x32x2f32(rx[((S_) + kw) % D][kh], ry[S_], acc[kh * 3 + kw], 0, 0, 0); \
        }
#pragma unroll
        for (int d = 0; d < D; ++d) W32_LOAD(d, d)
        int t = 0;
        for (; t + D <= S; t += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) { W32_MMA(d) W32_LOAD(d, t + D + d) }
        }
        // (the last, partial trip also needs X of the two positions behind it)
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (t + d < S) { W32_MMA(d) W32_LOAD(d, t + D + d) }
#undef W32_LOAD
#undef W32_MMA
    }
    float* redb = red + 4 * 9 * 32 * 32;
    bsum += __shfl_xor(bsum, 32, 64);
    if (lhi == 0) redb[wave * 32 + l32] = bsum;
    wgrad_reduce_store(acc, red, a.dW + (size_t)split * a.split_stride, o0, i0, a.cout, a.cin);
    if (i0 == 0 && tid < 32 && o0 + tid < a.cout)
        a.db[(size_t)split * a.split_stride + o0 + tid] = ((redb[tid] + redb[32 + tid]) + redb[64 + tid]) + redb[96 + tid];
}

static Wgrad32Args wgrad_f32_args(const Plan& p, const float* dY, const float* X, float* dW, float* db, int cin, int cout, int splits)
{
    Wgrad32Args a;
    a.dY = dY; a.X = X; a.dW = dW; a.db = db; a.split_stride = p.grad_stride;
    a.cin = cin; a.cout = cout; a.GX = cdiv(cin, 8); a.GY = cdiv(cout, 8);
    a.PP = p.g.padded_positions(); a.PPT = p.PPT; a.guard = p.guard; a.Wp = p.g.Wp;
    a.len = cdiv(a.PP, splits * 4 * 8) * 8;
    a.o_tiles = cdiv(cout, 32); a.i_tiles = cdiv(cin, 32); a.splits = splits;
    a.items_per_xcd = cdiv(a.o_tiles * a.i_tiles * splits, 8);
    return a;
}

// ------------------------------------------------------------------ classifier backward
//   g = d loss / d z from the loss kernel's slots (gather_g), also left in gz;
//   da2[p][o] = [a2[p][o] > 0] * sum_c g[c][p] * W3[c][o];   dW3, db3: one slot per block (the optimiser kernel adds them)
// A block of 256 threads takes 64 padded positions.  Bound by its chain of dependent memory round
// trips, like the bfloat16 kernel of the same layer.
// (Four wavefronts for da2 and four for dW3 side by side, as there: without prefetching what a role reads,
// 16 x 16 cells 203 -> 208 us and 68 x 120 cells 901 -> 911 us a call; with it 203 -> 197 and 900 -> 893, but at
// 204 registers, one block per compute unit.)
constexpr int B32_BP = 64;

__global__ void __launch_bounds__(256)
k_conv3_bwd_f32(const float* __restrict__ slots, const float* __restrict__ T, const unsigned long long* __restrict__ n_valid,
                int CP, LossTiling lt, const float* __restrict__ a2, const float* __restrict__ W3T, float* __restrict__ da2,
                float* __restrict__ gz, float* __restrict__ part, Geo g, int PPT, int guard)
{
    constexpr int BP = B32_BP, GP = BP + 8;     // (pitch: the two halves of a B read 32 banks apart)
    __shared__ __attribute__((aligned(16))) float g_cp[32 * GP];    // [class][position]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int PP = g.padded_positions(), hw = g.h * g.w;
    const int m0 = blockIdx.x * BP;
    {
        const int pl = tid & 63, cq = tid >> 6;
        float v[8];
        const GatherCell cell = gather_g<8, 4>(slots, T, n_valid[0], CP, lt, g, m0 + pl, PP, cq, v);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int c = cq + 4 * k;
            g_cp[c * GP + pl] = c < g.C ? v[k] : 0.f;
            if (c < g.C && cell.inside) gz[((size_t)cell.img * g.C + c) * hw + cell.cy * g.w + cell.cx] = v[k];
        }
    }
    __syncthreads();

    const int OT = (g.c2 + 31) / 32, G2 = (g.c2 + 7) / 8, CG = (g.C + 7) / 8;
    {
        const int pm = (wave & 1) * 32 + l32, mp = m0 + pm;
        float gb[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) gb[q][e] = g_cp[(q * 8 + lhi * 4 + e) * GP + pm];
        for (int t = wave >> 1; t < OT; t += 2) {
            f32x4 wf[4], mk[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) wf[q] = *(const f32x4*)(W3T + ((t * 4 + q) * 64 + lane) * 4);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mk[q] = *(const f32x4*)(a2 + ((size_t)min(t * 4 + q, G2 - 1) * PPT + guard + min(mp, PP - 1)) * 8 + lhi * 4);
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < CG)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[q][e], gb[q][e], acc, 0, 0, 0);
            // (g is zero on the border, and so is da2)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t * 4 + q < G2 && mp < PP) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = mk[q][e] > 0.f ? acc[q * 4 + e] : 0.f;
                    *(f32x4*)(da2 + ((size_t)(t * 4 + q) * PPT + guard + mp) * 8 + lhi * 4) = v;
                }
        }
    }
    // dW3: k = positions, the two halves of the block's 64
    float* slot = part + (size_t)blockIdx.x * (32 * g.k2 + 32);
    f32x4 ga[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) ga[q] = *(const f32x4*)(g_cp + l32 * GP + lhi * 32 + q * 4);
    for (int t = wave; t < OT; t += 4) {
        const float* ab = a2 + (size_t)min((t * 32 + l32) >> 3, G2 - 1) * PPT * 8 + (l32 & 7);
        float av[32];
#pragma unroll
        for (int s = 0; s < 32; ++s) av[s] = ab[(size_t)(guard + min(m0 + lhi * 32 + s, PP - 1)) * 8];
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < 32; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ga[s >> 2][s & 3], av[s], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int c = (r >> 2) * 8 + lhi * 4 + (r & 3);
            if (c < g.C && t * 32 + l32 < g.k2) slot[c * g.k2 + t * 32 + l32] = acc[r];
        }
    }
    {   // db3: eight threads per class
        const int c = tid >> 3, q = tid & 7;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += g_cp[c * GP + q * 8 + k];
        s += __shfl_xor(s, 1, 64); s += __shfl_xor(s, 2, 64); s += __shfl_xor(s, 4, 64);
        if (q == 0 && c < g.C) slot[32 * g.k2 + c] = s;
    }
}

// ------------------------------------------------------------------ host-side entry points
void forward_f32(Ctx& c, const Plan& p, char* ws)
{
    const Geo& g = p.g;
    auto f = [&](size_t at) { return at ? (float*)(ws + at) : nullptr; };
    conv_f32(c, "conv1_fwd_f32", p, 0, f(p.feat), f(p.wq1), g.c_in, g.c1, f(p.bq1), nullptr, f(p.a1), nullptr, nullptr, nullptr);
    conv_f32(c, "conv2_fwd_logits_f32", p, 2, f(p.a1), f(p.wq2), g.c1, g.c2, f(p.bq2), nullptr, f(p.a2), f(p.wq3), f(p.zpart), nullptr);
}

void backward_f32(Ctx& c, const Plan& p, char* ws, float* dfeat)
{
    const Geo& g = p.g;
    auto f = [&](size_t at) { return (float*)(ws + at); };
    ST_LAUNCH(c, "conv3_bwd_f32", k_conv3_bwd_f32, dim3(p.blocks3), dim3(256), 0, f(p.g_slots), f(p.tadj),
              (const unsigned long long*)(ws + p.counters), (g.C + 3) / 4 * 4, p.lt, f(p.a2), f(p.wq3t), f(p.da2), f(p.gz), f(p.grad3), g,
              p.PPT, p.guard);
    conv_f32(c, "conv2_dgrad_f32", p, 1, f(p.da2), f(p.wq2t), g.c2, g.c1, nullptr, f(p.a1), f(p.da1), nullptr, nullptr, nullptr);
    if (dfeat)
        conv_f32(c, "conv1_dgrad_f32", p, 3, f(p.da1), f(p.wq1t), g.c1, g.c_in, nullptr, nullptr, nullptr, nullptr, nullptr, dfeat);
    float* grad = f(p.grad);
    const Wgrad32Args a1 = wgrad_f32_args(p, f(p.da1), f(p.feat), grad + p.po.W1, grad + p.po.b1, g.c_in, g.c1, p.splits1);
    const Wgrad32Args a2 = wgrad_f32_args(p, f(p.da2), f(p.a1), grad + p.po.W2, grad + p.po.b2, g.c1, g.c2, p.splits2);
    const int blocks1 = a1.items_per_xcd * 8, blocks2 = a2.items_per_xcd * 8;
    ensure_dynamic_lds((const void*)k_wgrad3x3_f32, WGRAD_SMEM_BYTES);
    ST_LAUNCH(c, "conv12_wgrad_f32", k_wgrad3x3_f32, dim3(blocks1 + blocks2), dim3(256), WGRAD_SMEM_BYTES, a1, a2, blocks1);
}

}  // namespace st
