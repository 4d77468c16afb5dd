// Float32 path: the head's 3x3 contractions on the bfloat16 matrix cores with float32 operands kept whole.  (The convolutions of grids
// with few tiles and the weight gradients of small frames on the float32 instruction: k_conv3x3_f32_few, k_wgrad3x3_f32_few.)
//
// A float32 value from 2^-110 to 3.39e38 is the exact sum of three bfloat16 values, each the rest of the ones before it rounded to nearest:
// x = xh + xm + xl.  Of the nine products of two such sums the six largest are formed,
//     xh wh  +  (xh wm + xm wh + xm wm + xh wl + xl wh),
// each exactly, and added in float32; what is left out is below 2^-24 of a product (worst 1.98 * 2^-25, at 1.0039 * 1.0039; root mean
// square over all mantissas 2^-27.5), of either sign.  (Cut off instead of rounded, the three parts have one sign, and what is left out
// shifts every sum the same way: weight gradients were three times further from float64 than the float32 instructions' for it.)  Six v_mfma_f32_32x32x16_bf16 take 192 cycles
// for what eight v_mfma_f32_32x32x2_f32 x 64 cycles do.  Errors against float64 (2-norm, seven sizes from 16 x 16 cells
// and 24 channels to 140 x 250 and 256, four seeds each): logits 1.1 - 1.8e-7 (1.5 - 3.8e-7 with the float32 instructions), feature
// gradient 1.5 - 2.0e-7 (1.9 - 3.4e-7); weight gradients: see there.
// Measured, 68 x 120 cells, 256 -> 128 -> 128, us per launch, float32 instructions / here: layer 1 49.6 / 36, layer 2 with the
// classifier 28.3 / 23.5, its data gradient 27.2 / 22, weight gradients 77 / 49; a 4-step call 901 -> 686, 16 x 16 cells unchanged.
// What binds now: a wavefront issues one instruction in four cycles, and splitting (eleven per pair of values) leaves few of
// the eight places an MFMA takes empty -- about 7.5 are used.
//
// The whole range of float32.  A bfloat16 has no bits below 2^-133, so the last parts of a value below 2^-110 would be lost.
// Operands therefore enter times 2^24 -- weights from the kernel that writes their copies, activations on their way to LDS, both operands
// of a weight gradient as they are split -- which puts
// even the last bit of a subnormal, 2^-149, among the normal values, and the sums are taken times 2^-48.  What that makes overflow (an
// operand from 2^104 or a sum from 2^80 on), infinities and NaN give sums that are not finite: those are formed again, from the
// operands as they are, by the float32 instruction (conv_f32_plain, wgrad_f32_plain), and no others.  Factors and test cost the
// convolutions 0.5 % of the 68 x 120 call (659 -> 662 us).
//
// Everything stays float32 in memory -- activations in runs of eight channels [c / 8][position][8] (pos8_index), weights in the
// fragment order of wfrag_index -- and is split by the kernel that reads it, between its MFMAs.  (Weights written as three
// planes by the optimiser kernel made that kernel slower by more than the splitting costs: 7.6 -> 10.3 us at 256 -> 128 -> 128.)
#include <algorithm>
#include <utility>

#include "st_gather.hpp"
#include "st_kernels.hpp"
#include "st_mfma.hpp"
#include "st_wgrad.hpp"

namespace st {

#define CF_F __builtin_amdgcn_sched_barrier(0);

// f(0), f(1), .. f(N - 1) with the index as a constant expression
template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) { unrolled(f, std::make_integer_sequence<int, N>{}); }

// two values as bfloat16, to nearest even, and back
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned round_pair(float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2)); }
__device__ __forceinline__ float low_of(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float high_of(unsigned p) { return __builtin_bit_cast(float, p & 0xFFFF0000u); }

__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// ------------------------------------------------------------------ 3x3 convolution
//   out[p][n] = epi( sum_{tap, c} X[p + shift(tap)][c] * W[n][tap][c] )        p: padded positions
// A block is four wavefronts and owns 32 P positions x 32 output channels.  The K loop walks stages of (one kernel row) x (64
// input channels); of a stage each wavefront takes 16 channels, its partial sums are added through LDS in ascending order.
// A stage's activations (32 P + 2 positions) come as float32 into registers a stage ahead, are split between the MFMAs of the
// stage before and go to LDS as three planes of 128-byte rows, 16-byte chunk c of row r at c ^ ((r >> 1) & 7); two such slabs
// alternate.  Per tap a wavefront reads 3 P fragments of 1 KB from LDS and 2 KB of weights for 6 P MFMAs, so neither
// path is near its limit.  P is chosen so that the blocks fill whole rounds of the chip (conv_split_p): 68 x 120 cells and
// 128 channels are 1120 tiles of 32 x 32, 4.4 per compute unit, which 224 blocks of five tiles take in one round.
// (Tried, the same shape, layer 1: three tiles and two blocks per compute unit 40 us; two accumulators for the small products
// instead of one 38; fragments read one group ahead and the barrier behind the last group 37.)
struct Conv32Args {
    const float* X;       // pos8 layout, G groups of eight channels
    const float* Wf;      // fragment order (wfrag_index, k = 8 G), rows = output channels; scaled for the split kernel
    const float* bias;    // EPI 0, 2: zeros behind the last channel
    const float* mask;    // EPI 1: activation whose sign gates the gradient (layout of Y)
    float* Y;             // pos8 layout, GY groups (EPI 2: may be null)
    const float* W3f;     // EPI 2: [32 classes][w3_pitch], zero beyond the classes and channels
    float* zpart;         // EPI 2: this channel tile's share of the logits, [n-tile][padded position][zpitch]
    float* dense;         // EPI 3: [n][dense_c][h][w]
    int PP, Hp, Wp, h, w, G, GY, PPT, guard, w3_pitch, zpitch, dense_c;
    int m_tiles, n_tiles, tiles_per_xcd;
    // the weights as they are: element (row, tap, k) at row * w_row + tap * w_tap + k * w_k.  (Behind what every block reads first.)
    int rows, K, w_row, w_tap, w_k;
    const float* W;
};

template <int P>
constexpr size_t conv_split_lds()
{
    return std::max((size_t)2 * 3 * (32 * P + 2) * 128, (size_t)4 * P * 4096);     // slabs; partial sums
}

// Of the share of a block's sums that wavefront `wave` has, those that are not finite, formed by the float32 matrix instruction
// (v_mfma_f32_32x32x2_f32; number e of 16 channels pairs channel e with channel 8 + e).
template <int P>
__device__ __forceinline__ void conv_f32_plain(const Conv32Args& a, int m0, int nt, int wave, f32x16 (&acc)[P])
{
    const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5, row = nt * 32 + l32;
    f32x16 sum[P];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[j][r] = 0.f;
#pragma unroll 1
    for (int c0 = wave * 2; c0 < a.G; c0 += 8) {
        const int run = c0 + lhi;
#pragma unroll 1
        for (int tap = 0; tap < 9; ++tap) {
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = run * 8 + e;
                w[e] = row < a.rows && k < a.K ? a.W[row * a.w_row + tap * a.w_tap + k * a.w_k] : 0.f;
            }
            // (a run that does not exist: zeros, from the guard in front of the first)
            const float* xp = run < a.G ? a.X + ((ptrdiff_t)run * a.PPT + a.guard + m0 + l32 + (tap / 3 - 1) * a.Wp + tap % 3 - 1) * 8 : a.X;
            const int step = run < a.G ? 256 : 0;
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const f32x4 x0 = *(const f32x4*)(xp + j * step), x1 = *(const f32x4*)(xp + j * step + 4);
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], e < 4 ? x0[e & 3] : x1[e & 3], sum[j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = __builtin_isfinite(acc[j][r]) ? acc[j][r] : sum[j][r];
}

// Closes a block's tile of 32 P positions x 32 channels: the sums of its KG wavefronts are added through LDS in ascending order (red:
// [wavefront][P][4 register groups][64 lanes][4]), and the first four finish a quarter of the channels each.
template <int EPI, int P, int KG>
__device__ __forceinline__ void conv_f32_finish(const Conv32Args& a, int m0, int nt, float* red, f32x16 (&acc)[P])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    // ---- what the epilogue needs from memory, on its way while the sums are exchanged
    const int rq = wave, ct = rq * 8 + lhi * 4, ch = nt * 32 + ct;      // this lane's 4 channels
    const bool ends = KG == 4 || wave < 4;
    f32x4 bias = {0.f, 0.f, 0.f, 0.f}, w3 = {0.f, 0.f, 0.f, 0.f}, mask[EPI == 1 ? P : 1];
    if (ends && (EPI == 0 || EPI == 2)) bias = *(const f32x4*)(a.bias + ch);
    if (ends && EPI == 2) w3 = *(const f32x4*)(a.W3f + (size_t)l32 * a.w3_pitch + ch);
    const int run_out = min(nt * 4 + rq, a.GY - 1);
    if (ends && EPI == 1) {
#pragma unroll
        for (int j = 0; j < P; ++j) mask[j] = *(const f32x4*)(a.mask + ((size_t)run_out * a.PPT + a.guard + min(m0 + j * 32 + l32, a.PP - 1)) * 8 + lhi * 4);
    }

    // ---- partial sums of the wavefronts
    __syncthreads();
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            const f32x4 v = {acc[j][rq * 4], acc[j][rq * 4 + 1], acc[j][rq * 4 + 2], acc[j][rq * 4 + 3]};
            *(f32x4*)(red + (((wave * P + j) * 4 + rq) * 64 + lane) * 4) = v;
        }
    __syncthreads();

    // wavefront rq finishes channels 8 rq .. + 7 of the tile: a lane holds 4 channels of one position per 32 positions
    const int frame = a.Hp * a.Wp;
    f32x4 out[P];
    if (ends)
#pragma unroll
    for (int j = 0; j < P; ++j) {
        const int mp = m0 + j * 32 + l32;
        const int img = mp / frame, rr = mp - img * frame, y = rr / a.Wp, x = rr - y * a.Wp;
        const bool inside = mp < a.PP && y >= 1 && y <= a.h && x >= 1 && x <= a.w;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KG; ++k) v += *(const f32x4*)(red + (((k * P + j) * 4 + rq) * 64 + lane) * 4);
        const size_t at = ((size_t)(nt * 4 + rq) * a.PPT + a.guard + mp) * 8 + lhi * 4;
        const bool stored = nt * 4 + rq < a.GY && mp < a.PP;
        if (EPI == 0 || EPI == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = inside ? fmaxf(v[e] + bias[e], 0.f) : 0.f;
        } else if (EPI == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = inside && mask[j][e] > 0.f ? v[e] : 0.f;
        }
        if (EPI == 3) {
            if (inside) {
                float* dst = a.dense + (((size_t)img * a.dense_c + ch) * a.h + (y - 1)) * a.w + (x - 1);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ch + e < a.dense_c) dst[(size_t)e * a.h * a.w] = v[e];
            }
        } else if (stored && a.Y) *(f32x4*)(a.Y + at) = v;
        out[j] = v;
    }
    if (EPI == 2) {
        // the classifier rides along: what this lane holds is the B operand of four float32 MFMAs
        // (v_mfma_f32_32x32x2_f32) against W3 (rows = classes, k = the 8 channels of this wavefront); the four
        // wavefronts' sums meet in LDS.  (All shares of the logits: one per 32 channels.)
        __syncthreads();       // the partial sums are read
        if (ends)
#pragma unroll
        for (int j = 0; j < P; ++j) {
            f32x16 z;
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_32x32x2f32(w3[e], out[j][e], z, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4*)(red + (((rq * P + j) * 4 + q) * 64 + lane) * 4) = f32x4{z[q * 4], z[q * 4 + 1], z[q * 4 + 2], z[q * 4 + 3]};
        }
        __syncthreads();
        if (ends && rq * 8 + lhi * 4 < a.zpitch) {     // (here rq: classes 8 rq .. + 7)
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const int mp = m0 + j * 32 + l32;
                f32x4 t = *(const f32x4*)(red + ((j * 4 + rq) * 64 + lane) * 4);
#pragma unroll
                for (int k = 1; k < 4; ++k) t += *(const f32x4*)(red + (((k * P + j) * 4 + rq) * 64 + lane) * 4);
                if (mp < a.PP) *(f32x4*)(a.zpart + ((size_t)nt * a.PP + mp) * a.zpitch + rq * 8 + lhi * 4) = t;
            }
        }
    }
}

template <int EPI, int P>
__global__ void __launch_bounds__(256, P <= 2 ? 2 : 1) k_conv3x3_f32(Conv32Args a)
{
    constexpr int BM = 32 * P, PLANE = (BM + 2) * 128, SLAB = 3 * PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // (consecutive blocks go to different XCDs: every XCD gets a contiguous run of position tiles)
    const int tile = (blockIdx.x % 8) * a.tiles_per_xcd + blockIdx.x / 8;
    if ((int)(blockIdx.x / 8) >= a.tiles_per_xcd || tile >= a.m_tiles * a.n_tiles) return;
    const int mt = tile / a.n_tiles, nt = tile % a.n_tiles;
    const int m0 = mt * BM;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;

    f32x16 acc[P], rest[P];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[j][r] = 0.f; rest[j][r] = 0.f; }

    const int c_chunks = (a.G + 7) >> 3, n_stages = 3 * c_chunks;

    // ---- activations: a unit is one position x one run of eight channels.  Unit u of a thread is number u * 256 + tid, counted
    // along the positions first; unit P is one of the 16 units of the last two positions (sixteen threads do the same one).
    int run[P + 1], row[P + 1];
#pragma unroll
    for (int u = 0; u < P; ++u) { const int q = u * 256 + tid; run[u] = q / BM; row[u] = q - run[u] * BM; }
    run[P] = (tid >> 1) & 7; row[P] = BM + (tid & 1);
    int lds_at[P + 1];
#pragma unroll
    for (int u = 0; u <= P; ++u) lds_at[u] = row[u] * 128 + ((run[u] ^ ((row[u] >> 1) & 7)) << 4);
    // (rows behind the grid lie in the guard, whose length counts on tiles of at most 256 positions)
    static_assert(BM <= 256, "guard rows");
    const float* xs = a.X + ((ptrdiff_t)a.guard + m0 - 1 - a.Wp) * 8;      // the stage on its way to the registers
    int x_cc = 0;
    f32x4 xr[P + 1][2];
    // (runs behind the last one: zeros, from the guard in front of the first)
    auto load_unit = [&](int u) __attribute__((always_inline)) {
        const float* src = x_cc * 8 + run[u] < a.G ? xs + ((size_t)run[u] * a.PPT + row[u]) * 8 : a.X;
        xr[u][0] = *(const f32x4*)src;
        xr[u][1] = *(const f32x4*)(src + 4);
    };
    // A unit's splitting and its three LDS writes, in steps that go between MFMAs: pair e (0 .. 3) of the eight values in one
    // step or in two, then plane by plane.
    u32x4 xp[3];
    float r0 = 0.f, r1 = 0.f;
    auto scale = [&](int u, int e) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) xr[u][e >> 1][(e & 1) * 2 + i] *= F32_SPLIT_SCALE;
    };
    auto split_a = [&](int u, int e) __attribute__((always_inline)) {
        const float v0 = xr[u][e >> 1][(e & 1) * 2], v1 = xr[u][e >> 1][(e & 1) * 2 + 1];
        const unsigned h = round_pair(v0, v1);
        xp[0][e] = h;
        r0 = __fsub_rn(v0, low_of(h)); r1 = __fsub_rn(v1, high_of(h));
    };
    auto split_b = [&](int e) __attribute__((always_inline)) {
        const unsigned m = round_pair(r0, r1);
        xp[1][e] = m;
        xp[2][e] = round_pair(__fsub_rn(r0, low_of(m)), __fsub_rn(r1, high_of(m)));
    };
    auto write_plane = [&](int u, int slab, int q) __attribute__((always_inline)) {
        *(u32x4*)(smem + slab * SLAB + q * PLANE + lds_at[u]) = xp[q];
    };
    // stages run over the channels first, then over the kernel rows
    auto x_next = [&]() __attribute__((always_inline)) {
        if (++x_cc == c_chunks) { x_cc = 0; xs += (ptrdiff_t)a.Wp * 8 - (ptrdiff_t)(c_chunks - 1) * 8 * a.PPT * 8; }
        else xs += (ptrdiff_t)8 * a.PPT * 8;
    };

    // ---- weights of this wavefront's 16 channels: per tap of a stage eight float32 values per lane (row l32, k 8 lhi ..), split
    // into three fragments.  While the matrix cores work on one tap the fragments of the tap before it are made for the
    // next stage (while they work on the first tap: those of the last tap, for this stage), a few instructions at a time.
    const float* wp = a.Wf + ((size_t)nt * 9 * a.G + wave * 2) * 256 + lane * 8;
    const size_t w_tap = (size_t)a.G * 256;
    int w_cc = 0;
    f32x4 wr[3][2];
    u32x4 wa[3][3];
    // (lanes whose channels do not exist: zeros, as above)
    auto load_w = [&](int kw) __attribute__((always_inline)) {
        const float* src = w_cc * 8 + wave * 2 + lhi < a.G ? wp + kw * w_tap : a.X + lane * 8;
        wr[kw][0] = *(const f32x4*)src;
        wr[kw][1] = *(const f32x4*)(src + 4);
    };
    auto w_next = [&]() __attribute__((always_inline)) {
        if (++w_cc == c_chunks) { w_cc = 0; wp += 3 * w_tap - (size_t)(c_chunks - 1) * 4 * 512; } else wp += 4 * 512;
    };
    float w0 = 0.f, w1 = 0.f, w2 = 0.f;
    auto split_w = [&](int kw, int i) __attribute__((always_inline)) {       // i: 0 .. 15, pair i / 4
        const int e = i >> 2;
        const float v0 = wr[kw][e >> 1][(e & 1) * 2], v1 = wr[kw][e >> 1][(e & 1) * 2 + 1];
        if ((i & 3) == 0) { wa[kw][0][e] = round_pair(v0, v1); w0 = __fsub_rn(v0, low_of(wa[kw][0][e])); }
        if ((i & 3) == 1) w1 = __fsub_rn(v1, high_of(wa[kw][0][e]));
        if ((i & 3) == 2) { wa[kw][1][e] = round_pair(w0, w1); w2 = __fsub_rn(w0, low_of(wa[kw][1][e])); }
        if ((i & 3) == 3) wa[kw][2][e] = round_pair(w2, __fsub_rn(w1, high_of(wa[kw][1][e])));
    };

    int rd[3];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) rd[kw] = (l32 + kw) * 128 + (((wave * 2 + lhi) ^ (((l32 + kw) >> 1) & 7)) << 4);
    // fragments of three groups (group g of a stage: tap g / P, positions 32 (g % P) ..) rotate: two groups ahead
    u32x4 xb[3][3];
    auto read_x = [&](int slab, int g, int q) __attribute__((always_inline)) {
        xb[g % 3][q] = *(const u32x4*)(smem + slab * SLAB + q * PLANE + rd[g / P] + (g % P) * 4096);
    };

    // ---- first stage into slab 0, second into the registers
#pragma unroll
    for (int u = 0; u <= P; ++u) load_unit(u);
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) load_w(kw);
    w_next();
    x_next();
#pragma unroll
    for (int u = 0; u <= P; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { scale(u, e); split_a(u, e); split_b(e); }
#pragma unroll
        for (int q = 0; q < 3; ++q) write_plane(u, 0, q);
        load_unit(u);
    }
#pragma unroll
    for (int kw = 0; kw < 2; ++kw) {
#pragma unroll
        for (int i = 0; i < 16; ++i) split_w(kw, i);
        load_w(kw);
    }
    __syncthreads();
    constexpr int AHEAD = P > 1 ? 2 : 3;           // groups of the next stage whose fragments are read before it begins (P == 1: all, then)
    if (P > 1)
#pragma unroll
        for (int g = 0; g < AHEAD; ++g)
#pragma unroll
            for (int q = 0; q < 3; ++q) read_x(0, g, q);

    // One stage out of slab B.  NEXT: another stage follows, whose activations wait in the registers; LOAD: and one behind
    // it, which x_next has been moved to.  Everything has its place between two MFMAs, in a pinned order; the barrier stands in front
    // of the last two groups, during which the next stage's first fragments are read.
    auto stage = [&](int B, auto NEXT_, auto LOAD_) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(NEXT_)::value, LOAD = decltype(LOAD_)::value;
        constexpr int PLACES = 18 * P, BAR = P > 1 ? PLACES - 12 : PLACES;      // the barrier: in front of this place
        constexpr int PER = BAR / (P + 1);             // places per unit: P = 1 .. 5: 9, 8, 10, 12, 13
        constexpr bool FINE = PER >= 12;               // a pair's splitting in two places
        constexpr int W0 = FINE ? 8 : 4;               // first place of the LDS writes, one per plane; the loads come behind them
        static_assert(P * PER + W0 + 3 <= BAR && W0 + 4 <= PER, "a unit's steps fit, all writes lie before the barrier");
        if (P == 1) {
#pragma unroll
            for (int g = 0; g < 3; ++g)
#pragma unroll
                for (int q = 0; q < 3; ++q) read_x(B, g, q);
        }
        CF_F
        unrolled<PLACES>([&](auto at_) __attribute__((always_inline)) {
            constexpr int at = decltype(at_)::value, g = at / 6, q = at % 6;
            constexpr int kw = g / P, j = g % P, b = g % 3, in_tap = j * 6 + q, wk = (kw + 2) % 3;
            if constexpr (NEXT && P > 1 && at == BAR) { __syncthreads(); CF_F }
            if constexpr (q == 0) acc[j] = mfma_bf16(wa[kw][0], xb[b][0], acc[j]);
            else rest[j] = mfma_bf16(wa[kw][q == 1 ? 2 : q == 2 || q == 4 ? 0 : 1], xb[b][q == 1 || q == 5 ? 0 : q == 2 ? 2 : 1], rest[j]);
            CF_F
            if constexpr (P > 1 && q < 3) {
                if constexpr (g + 2 < 3 * P) read_x(B, g + 2, q == 0 ? 0 : 3 - q);
                else if constexpr (NEXT) read_x(1 - B, g + 2 - 3 * P, q == 0 ? 0 : 3 - q);
            }
            if constexpr (NEXT && at / PER <= P) {
                constexpr int u = at / PER, v = at % PER;
                // (from three units on each is scaled while the one before it is written, the first, and shorter stages', when split)
                if constexpr ((u == 0 || P <= 2) && v < W0 && !(FINE && v & 1)) scale(u, FINE ? v >> 1 : v);
                if constexpr (P > 2 && u < P && v >= W0 && v < W0 + 4) scale(u + 1, v - W0);
                if constexpr (FINE && v < 8) { if constexpr (v & 1) split_b(v >> 1); else split_a(u, v >> 1); }
                if constexpr (!FINE && v < 4) { split_a(u, v); split_b(v); }
                if constexpr (v >= W0 && v < W0 + 3) write_plane(u, 1 - B, v - W0);
                if constexpr (LOAD && v == W0 + 3) load_unit(u);
            }
            if constexpr (kw == 0 || NEXT) {
#pragma unroll
                for (int i = in_tap * 16 / (6 * P); i < (in_tap + 1) * 16 / (6 * P); ++i) split_w(wk, i);
                // (of the next stage the last tap, of the one behind it the other two)
                if constexpr (in_tap == 6 * P - 1) {
                    if constexpr (kw == 0 ? NEXT : LOAD) load_w(wk);
                    if constexpr (NEXT && kw == 0) w_next();
                }
            }
            CF_F
        });
        if (NEXT && P == 1) __syncthreads();
    };
    const std::true_type yes; const std::false_type no;
    int s = 0;
    for (; s + 2 < n_stages; ++s) {
        x_next();
        stage(s & 1, yes, yes);
    }
    stage(s & 1, yes, no);
    stage((s + 1) & 1, no, no);

    // ---- the wavefront's sums, formed again where they are not finite
    float finite = 0.f;
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[j][r] = (acc[j][r] + rest[j][r]) * F32_SPLIT_BACK;
            finite = __builtin_fmaf(acc[j][r], 0.f, finite);
        }
    if (__builtin_expect(__ballot(finite != 0.f) != 0, 0)) conv_f32_plain<P>(a, m0, nt, wave, acc);

    conv_f32_finish<EPI, P, 4>(a, m0, nt, (float*)smem, acc);
}

// The same by the float32 instruction, for grids whose tiles of 32 x 32 leave compute units without a block.  There a launch is as long as
// one block's chain of steps, and sixteen wavefronts that split taps x runs of eight channels, operands straight from memory
// (lane l: row or position l % 32, channels 4 (l / 32) .. + 3 of a run, the four pairs of k that four MFMAs take), have a shorter one
// than four that hand split operands through LDS.
constexpr int CF_KG = 16, CF_DEPTH = 4;    // wavefronts; operand sets on their way per wavefront

template <int EPI>
__global__ void __launch_bounds__(64 * CF_KG) k_conv3x3_f32_few(Conv32Args a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // (the arguments in one trip: left to itself the compiler asks for them in four, one behind the other)
    asm volatile("" ::"s"(a.tiles_per_xcd), "s"(a.m_tiles), "s"(a.n_tiles), "s"(a.X), "s"(a.Wf), "s"(a.G), "s"(a.PPT), "s"(a.guard), "s"(a.Wp));
    const int tile = (blockIdx.x % 8) * a.tiles_per_xcd + blockIdx.x / 8;
    if ((int)(blockIdx.x / 8) >= a.tiles_per_xcd || tile >= a.m_tiles * a.n_tiles) return;
    const int mt = tile / a.n_tiles, nt = tile % a.n_tiles, m0 = mt * 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;

    f32x16 acc[1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = 0.f;

    const int total = 9 * a.G, per = (total + CF_KG - 1) / CF_KG;
    const int i0 = wave * per, i1 = min(total, i0 + per);
    if (i0 < i1) {
        const float* wp = a.Wf + ((size_t)nt * total + i0) * 256;            // advances by 256 per item
        const float* xb = a.X + (size_t)(a.guard + m0) * 8;
        const unsigned at = l32 * 8 + lhi * 4;
        int tap = i0 / a.G, g = i0 - tap * a.G, li = i0;
        const float* xp = xb + ((ptrdiff_t)g * a.PPT + (tap / 3 - 1) * a.Wp + (tap % 3 - 1)) * 8;
        f32x4 rw[CF_DEPTH], rx[CF_DEPTH];
        // (past the end of the run the last item is loaded again and not used)
        auto load = [&](int s) __attribute__((always_inline)) {
            rw[s] = *(const f32x4*)(wp + at);
            rx[s] = *(const f32x4*)(xp + at);
            if (++li < i1) {
                wp += 256;
                if (++g == a.G) {
                    g = 0; ++tap;
                    xp = xb + (ptrdiff_t)((tap / 3 - 1) * a.Wp + (tap % 3 - 1)) * 8;
                } else xp += (ptrdiff_t)a.PPT * 8;
            }
        };
        auto product = [&](int s) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(rw[s][e], rx[s][e], acc[0], 0, 0, 0);
        };
#pragma unroll
        for (int d = 0; d < CF_DEPTH; ++d) load(d);
        int i = i0;
        for (; i + CF_DEPTH <= i1; i += CF_DEPTH) {
#pragma unroll
            for (int d = 0; d < CF_DEPTH; ++d) { product(d); load(d); }
        }
#pragma unroll
        for (int d = 0; d < CF_DEPTH - 1; ++d)
            if (i + d < i1) product(d);
    }
    conv_f32_finish<EPI, 1, CF_KG>(a, m0, nt, (float*)smem, acc);
}

template <int EPI, int P>
static void conv_f32_launch(Ctx& c, const char* name, const Conv32Args& a)
{
    const size_t smem = conv_split_lds<P>();
    ensure_dynamic_lds((const void*)k_conv3x3_f32<EPI, P>, smem);
    ST_LAUNCH(c, name, (k_conv3x3_f32<EPI, P>), dim3(a.tiles_per_xcd * 8), dim3(256), smem, a);
}

// Tiles of 32 positions per block.  A layer's time goes with (blocks a compute unit gets) x (time of a block); the five block
// times are fitted to forward calls with each P forced, c -> c -> c channels, us for P = 1 .. 5:
//   30 x 50 cells, 128    28  33  39  43  49       68 x 120, 128    67  62  67  76  55
//   45 x 80, 128          46  44  41  45  51       80 x 140, 128    78  64  69  76  89
//   60 x 107, 128         57  48  66  47  53       90 x 160, 128    94  77  90  78  88
// (up to two tiles two blocks share a compute unit, which is why two small ones beat one large).  The float32 instructions'
// kernel: 27, 47, 56, 66, 76, 93 us.  One tile per block is for 64 input channels on few tiles (conv_f32_few).
static int conv_split_p(int m_units, int n_tiles)
{
    static const int block_time[5] = {16, 23, 35, 44, 55};
    int best = 1;
    long best_t = 0;
    for (int P = 1; P <= 5; ++P) {
        const long t = (long)cdiv((long long)cdiv(m_units, P) * n_tiles, 256) * block_time[P - 1];
        if (P == 1 || t < best_t) { best = P; best_t = t; }
    }
    return best;
}

// Whether a layer runs on k_conv3x3_f32_few: at most one tile of 32 x 32 per compute unit, and by the launches' times, which are
// 3.1 us + 0.44 per item of its wavefronts and, on split operands, 2.5 us + 0.83 per stage.  Only 57 - 64 input channels, whole
// stages of which a block walks three, are quicker split.  us per launch, few / split: 16 x 16 cells, 24 -> 32 channels 4.5 / 5.4, 64 -> 64
// 5.8 / 5.0, 128 -> 128 7.4 / 7.6, 256 -> 128 11.4 / 12.6; 30 x 50 cells, 320 -> 64 13.8 / 15.0; 45 x 80 cells, 64 -> 64 (260 tiles) 8.4 / 6.8.
// Calls of 4 steps, all split / as here: 16 x 16 cells, 24 -> 32 -> 24 202 / 190 us, 24 x 40, 256 -> 128 -> 128 305 / 297.
static bool conv_f32_few(const Geo& g, int cin, int cout)
{
    const int G = cdiv(cin, 8);
    if ((long long)cdiv(g.padded_positions(), 32) * cdiv(cout, 32) > 256) return false;
    return 310 + 44 * cdiv(9 * G, CF_KG) < 250 + 83 * 3 * cdiv(G, 8);
}
float conv_f32_weight_scale(const Geo& g, int cin, int cout) { return conv_f32_few(g, cin, cout) ? 1.f : F32_SPLIT_SCALE; }

// cin, cout: channels of the layer as run here (exchanged for a data gradient)
// W: that layer's weights, [o][tap][i] as its forward pass has them
static void conv_f32(Ctx& c, const char* name, const Plan& p, int epi, const float* X, const float* Wf, const float* W, int cin, int cout,
                     const float* bias, const float* mask, float* Y, const float* W3f, float* zpart, float* dense)
{
    const Geo& g = p.g;
    Conv32Args a;
    a.X = X; a.Wf = Wf; a.bias = bias; a.mask = mask; a.Y = Y; a.W3f = W3f; a.zpart = zpart; a.dense = dense;
    a.PP = g.padded_positions(); a.Hp = g.Hp; a.Wp = g.Wp; a.h = g.h; a.w = g.w;
    a.G = cdiv(cin, 8); a.GY = cdiv(cout, 8); a.PPT = p.PPT; a.guard = p.guard;
    a.w3_pitch = cdiv(g.c2, 32) * 32; a.zpitch = (g.C + 3) / 4 * 4; a.dense_c = cout;
    a.rows = cout; a.K = cin;
    const bool forward = epi == 0 || epi == 2;
    a.W = forward ? W : W + 8 * cout;        // (a data gradient has the taps mirrored)
    a.w_row = forward ? 9 * cin : 1; a.w_tap = forward ? cin : -cout; a.w_k = forward ? 1 : 9 * cout;
    a.n_tiles = cdiv(cout, 32);
    const bool few = conv_f32_few(g, cin, cout);
    const int P = few ? 1 : conv_split_p(cdiv(a.PP, 32), a.n_tiles);
    a.m_tiles = cdiv(a.PP, 32 * P);
    a.tiles_per_xcd = cdiv(a.m_tiles * a.n_tiles, 8);
    auto go = [&](auto e) {
        constexpr int E = decltype(e)::value;
        if (few) {
            const size_t smem = CF_KG * 4096;
            ensure_dynamic_lds((const void*)k_conv3x3_f32_few<E>, smem);
            ST_LAUNCH(c, name, k_conv3x3_f32_few<E>, dim3(a.tiles_per_xcd * 8), dim3(64 * CF_KG), smem, a);
            return;
        }
        switch (P) {
        case 1: conv_f32_launch<E, 1>(c, name, a); break;
        case 2: conv_f32_launch<E, 2>(c, name, a); break;
        case 3: conv_f32_launch<E, 3>(c, name, a); break;
        case 4: conv_f32_launch<E, 4>(c, name, a); break;
        default: conv_f32_launch<E, 5>(c, name, a); break;
        }
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
// One wavefront accumulates 32 (o) x 32 (i) x 9 (taps), k = 16 positions per unit.  A lane reads the eight positions of its
// channel that an operand needs as eight 4-byte loads and splits them itself.  As in the bfloat16 kernel dY is what moves by
// one position for the taps to the left and right: ten positions of it are read, and the three fragments of a plane are packed
// from them.  34 loads and some 270 vector instructions for 54 MFMAs (1728 cycles), all for units to come.
// (dY is zero on the border of the grid and in the guard.)
// The large products have accumulators of their own, as in the convolution.  An MFMA cuts off downwards what lies far below its
// accumulator, and six of them per unit into one round more often than eight float32 instructions do: error of the sums against
// float64 (2-norm, same dY and features, ten sizes from 16 x 16 cells and 24 channels to 140 x 250 and 128, six seeds each), float32
// instructions / six into one accumulator / here: 0.63 - 2.8e-7, mean 1.03 / 0.65 - 3.8e-7, mean 1.25, shifted by - 0.14 - 1.2e-7
// of the elements' size / 0.55 - 1.6e-7, mean 0.76, no shift.
// 18 tiles of accumulators leave 224 registers for operands; of X only one unit's fragments are held therefore, a kernel row at a time.
// Measured, 68 x 120 cells, 256 -> 128 -> 128: 77 us with the float32 instructions, 43.8 into one accumulator and without the factors, 49
// here; four steps 667 -> 686 us, 24 x 40 cells 311 -> 318, 90 x 160 cells, 128 channels 808 -> 828.  (One unit
// ahead instead of two, one loop body, cleared by MFMAs, the test behind the sum over the wavefronts: 685 - 692 us.)
// The rest (four wavefronts per block added through LDS, position splits added by the optimiser
// kernel, both layers in one launch) is as for the bfloat16 kernel.
struct Wgrad32Args {
    const float* dY; const float* X; float* dW; float* db;
    size_t split_stride;
    int cin, cout, GX, GY, PPT, guard, Wp, n_units, units_per_wave;       // units of 16 positions (k_wgrad3x3_f32_few: 8)
    int o_tiles, i_tiles, splits, items_per_xcd;
};

// Those of a wavefront's sums that are not finite, formed by the float32 matrix instruction (number e of a unit pairs positions e and 8 + e).
__device__ __forceinline__ void wgrad_f32_plain(const float* yp, const float* xp, ptrdiff_t xrow, int units, f32x16 (&acc)[9])
{
    f32x16 sum[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[t][r] = 0.f;
#pragma unroll 1
    for (int u = 0; u < units; ++u, yp += 128, xp += 128)
#pragma unroll 1
        for (int e = 0; e < 8; ++e) {
            float y[3], x[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) { y[k] = yp[(e + 1 - k) * 8]; x[k] = xp[(k - 1) * xrow + e * 8]; }
#pragma unroll
            for (int t = 0; t < 9; ++t) sum[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[t / 3], y[t % 3], sum[t], 0, 0, 0);
        }
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = __builtin_isfinite(acc[t][r]) ? acc[t][r] : sum[t][r];
}

__global__ void __launch_bounds__(256, 1) k_wgrad3x3_f32(Wgrad32Args a1, Wgrad32Args a2, int blocks1)
{
    extern __shared__ __attribute__((aligned(16))) float red[];
    const bool second = (int)blockIdx.x >= blocks1;
    const Wgrad32Args& a = second ? a2 : a1;
    const int bid = second ? blockIdx.x - blocks1 : blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = a.o_tiles * a.i_tiles;
    const int item = (bid % 8) * a.items_per_xcd + bid / 8;
    if (bid / 8 >= a.items_per_xcd || item >= tiles * a.splits) return;
    const int split = item / tiles, tile = item - split * tiles;
    const int o0 = (tile % a.o_tiles) * 32, i0 = (tile / a.o_tiles) * 32;

    f32x16 acc[9], rest[9];       // the large products' sums, and those of the other five
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[t][r] = 0.f; rest[t][r] = 0.f; }
    float bsum = 0.f;

    const int u0 = (split * 4 + wave) * a.units_per_wave, u1 = min(u0 + a.units_per_wave, a.n_units);
    if (u0 < u1) {
        // (channels beyond the last group re-read it: their sums are dropped at the end)
        auto operand = [&](const float* base, int c0, int runs, int lane) __attribute__((always_inline)) {
            const int l32 = lane & 31;
            return base + ((size_t)min((c0 + l32) >> 3, runs - 1) * a.PPT + a.guard + (size_t)u0 * 16 + (lane >> 5) * 8) * 8 + (l32 & 7);
        };
        const ptrdiff_t xrow = (ptrdiff_t)a.Wp * 8;
        // raw values of two units: positions - 1 .. 8 of dY, 0 .. 7 of X in the three rows
        float ry[2][10], rx[2][3][8];
        const float *yl = operand(a.dY, o0, a.GY, lane), *xl = operand(a.X, i0, a.GX, lane);        // the unit in work
        auto load_y = [&](int s, int ahead, int e) __attribute__((always_inline)) { ry[s][e] = yl[ahead * 128 + (e - 1) * 8]; };
        auto load_x = [&](int s, int ahead, int kh, int e) __attribute__((always_inline)) { rx[s][kh][e] = xl[(kh - 1) * xrow + ahead * 128 + e * 8]; };
        // Fragments: of dY for the unit in work and the next [dY at p + 1, p, p - 1][plane]; of X [kernel row][plane] for the unit in work,
        // each row replaced by the next unit's once its three taps are done
        u32x4 fy[2][3][3], fx[3][3];
        unsigned y4[3];
        float r0 = 0.f, r1 = 0.f;
        // dY: pairs of neighbouring positions 2 k - 1, 2 k (k = 0 .. 4), per plane; the fragment at p - 1 takes the first four, the one at
        // p + 1 the last four, the one at p the pairs between them
        auto put_y = [&](int s, int q, int k, unsigned v) __attribute__((always_inline)) { if (k < 4) fy[s][2][q][k] = v; else y4[q] = v; };
        auto split_ya = [&](int s, int k) __attribute__((always_inline)) {
            const float v0 = ry[s][2 * k] * F32_SPLIT_SCALE, v1 = ry[s][2 * k + 1] * F32_SPLIT_SCALE;
            const unsigned h = round_pair(v0, v1);
            put_y(s, 0, k, h);
            r0 = __fsub_rn(v0, low_of(h)); r1 = __fsub_rn(v1, high_of(h));
        };
        auto split_yb = [&](int s, int k) __attribute__((always_inline)) {
            const unsigned m = round_pair(r0, r1);
            put_y(s, 1, k, m);
            put_y(s, 2, k, round_pair(__fsub_rn(r0, low_of(m)), __fsub_rn(r1, high_of(m))));
        };
        auto place_y = [&](int s, int e) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const unsigned next = e < 3 ? fy[s][2][q][(e + 1) & 3] : y4[q];
                fy[s][1][q][e] = __builtin_amdgcn_alignbyte(next, fy[s][2][q][e], 2);
                fy[s][0][q][e] = next;
            }
        };
        auto split_xa = [&](int s, int kh, int e) __attribute__((always_inline)) {
            const float v0 = rx[s][kh][2 * e] * F32_SPLIT_SCALE, v1 = rx[s][kh][2 * e + 1] * F32_SPLIT_SCALE;
            const unsigned h = round_pair(v0, v1);
            fx[kh][0][e] = h;
            r0 = __fsub_rn(v0, low_of(h)); r1 = __fsub_rn(v1, high_of(h));
        };
        auto split_xb = [&](int kh, int e) __attribute__((always_inline)) {
            const unsigned m = round_pair(r0, r1);
            fx[kh][1][e] = m;
            fx[kh][2][e] = round_pair(__fsub_rn(r0, low_of(m)), __fsub_rn(r1, high_of(m)));
        };
        // What follows MFMA number t of a unit (18 per kernel row; raw values in slot S, the next unit's in N): the splitting of this unit's
        // last row, then of the next unit's dY and first two rows, and the loads that replace those raw values by the next but one's in
        // their slot.  (live: the next unit belongs to this wavefront's range)
        auto place = [&](auto N_, auto t_, bool live) __attribute__((always_inline)) {
            constexpr int N = decltype(N_)::value, S = 1 - N, t = decltype(t_)::value;
            constexpr int i = t < 8 ? t : t < 18 ? t - 8 : t < 26 ? t - 18 : t < 36 ? t - 26 : t < 44 ? t - 36 : t - 44;
            if constexpr (t < 8) { if constexpr (i & 1) split_xb(2, i >> 1); else split_xa(S, 2, i >> 1); }
            else if constexpr (t < 18) {
                if constexpr (i & 1) split_yb(N, i >> 1); else split_ya(N, i >> 1);
                if constexpr (i < 8) load_x(S, 2, 2, i);
            } else if constexpr (t < 26) { if constexpr (i & 1) split_xb(0, i >> 1); else split_xa(N, 0, i >> 1); }
            else if constexpr (t < 36) {
                if constexpr (i < 8) { bsum += live ? ry[N][i + 1] : 0.f; load_x(N, 3, 0, i); }
                load_y(N, 3, i);
            } else if constexpr (t < 44) { if constexpr (i & 1) split_xb(1, i >> 1); else split_xa(N, 1, i >> 1); }
            else {
                if constexpr (i < 8) load_x(N, 3, 1, i);
                if constexpr (i >= 6) place_y(N, i - 6);
            }
        };
        const std::integral_constant<int, 0> slot0; const std::integral_constant<int, 1> slot1;
        auto unit = [&](auto S_, bool next_live) __attribute__((always_inline)) {
            constexpr int S = decltype(S_)::value;
            unrolled<54>([&](auto t_) __attribute__((always_inline)) {
                constexpr int t = decltype(t_)::value, kh = t / 18, q = t % 18 / 3, kw = t % 3, tap = kh * 3 + kw;
                constexpr int px[6] = {2, 0, 1, 0, 1, 0}, py[6] = {0, 2, 1, 1, 0, 0};
                if constexpr (q == 5) acc[tap] = mfma_bf16(fx[kh][0], fy[S][kw][0], acc[tap]);
                else rest[tap] = mfma_bf16(fx[kh][px[q]], fy[S][kw][py[q]], rest[tap]);
                CF_F
                place(std::integral_constant<int, 1 - S>{}, t_, next_live);
                CF_F
            });
            yl += 128; xl += 128;
        };
        // (loads run up to three units past the end of the range: guard positions, not used)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int e = 0; e < 10; ++e) load_y(s, s, e);
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int e = 0; e < 8; ++e) load_x(s, s, kh, e);
        }
        asm volatile("" ::: "memory");
        // the first unit's dY and first two rows, as a unit in front of it would do it
        xl -= 128; yl -= 128;
        unrolled<46>([&](auto i_) __attribute__((always_inline)) { place(slot0, std::integral_constant<int, decltype(i_)::value + 8>{}, true); CF_F });
        xl += 128; yl += 128;
        int u = u0;
        for (; u + 2 <= u1; u += 2) {
            unit(slot0, true);
            asm volatile("" ::: "memory");
            unit(slot1, u + 2 < u1);
            asm volatile("" ::: "memory");
        }
        if (u < u1) unit(slot0, false);

        // ---- the sums, formed again where they are not finite
        float finite = 0.f;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[t][r] = (acc[t][r] + rest[t][r]) * F32_SPLIT_BACK;
                finite = __builtin_fmaf(acc[t][r], 0.f, finite);
            }
        if (__builtin_expect(__ballot(finite != 0.f) != 0, 0)) {
            // (Where the operands begin is found anew: kept over the loop it was kept in scratch memory, 52 bytes a lane.  68 x 120 cells, 256 -> 128 ->
            //  128 channels 663.7 -> 659.6 us a call of four steps, 135 x 240 cells, 64 channels 795.6 -> 791.9)
            int again = threadIdx.x & 63;
            asm volatile("" : "+v"(again));
            wgrad_f32_plain(operand(a.dY, o0, a.GY, again), operand(a.X, i0, a.GX, again), xrow, u1 - u0, acc);
        }
    }
    float* redb = red + 4 * 9 * 32 * 32;
    bsum += __shfl_xor(bsum, 32, 64);
    int tid2 = threadIdx.x;
    asm volatile("" : "+v"(tid2));       // (the same once more)
    if ((tid2 & 32) == 0) redb[(tid2 >> 6) * 32 + (tid2 & 31)] = bsum;
    wgrad_reduce_store<true>(acc, red, a.dW + (size_t)split * a.split_stride, o0, i0, a.cout, a.cin);
    if (i0 == 0 && tid2 < 32 && o0 + tid2 < a.cout)
        a.db[(size_t)split * a.split_stride + o0 + tid2] = ((redb[tid2] + redb[32 + tid2]) + redb[64 + tid2]) + redb[96 + tid2];
}

// The same by the float32 instruction, for frames that leave a wavefront few positions: there a launch is what comes before and behind the
// products, which is less here (no splitting, half the accumulators).  The two values of k of an MFMA are not neighbours but the
// same place in the two halves of the wavefront's range: a lane walks its half one position at a time, and the three taps of a kernel row
// are the values it holds for the previous, this and the next position.  Per position four 4-byte loads feed nine MFMAs.
__global__ void __launch_bounds__(256) k_wgrad3x3_f32_few(Wgrad32Args a1, Wgrad32Args a2, int blocks1)
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

    const int u0 = (split * 4 + wave) * a.units_per_wave, u1 = min(u0 + a.units_per_wave, a.n_units);
    const int half = (u1 - u0) * 4;          // (the positions are a multiple of eight)
    if (half > 0) {
        // (channels beyond the last group re-read it: their sums are dropped at the end)
        const size_t from = (size_t)a.guard + u0 * 8 + lhi * half;
        const float* yp = a.dY + ((size_t)min((o0 + l32) >> 3, a.GY - 1) * a.PPT + from) * 8 + (l32 & 7);
        const float* xp = a.X + ((size_t)min((i0 + l32) >> 3, a.GX - 1) * a.PPT + from) * 8 + (l32 & 7);
        // slot s of the ring holds dY of position s (mod 8) and X of position s - 1.  Loads run up to fifteen positions past the half
        // (guard positions make them readable).
        constexpr int D = 8;
        float ry[D], rx[D][3];
        auto load = [&](int s, int t) __attribute__((always_inline)) {
            ry[s] = yp[t * 8];
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) rx[s][kh] = xp[(t - 1 + (kh - 1) * a.Wp) * 8];
        };
        auto products = [&](int s) __attribute__((always_inline)) {
            bsum += ry[s];
#pragma unroll
            for (int k = 0; k < 9; ++k) acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(rx[(s + k % 3) % D][k / 3], ry[s], acc[k], 0, 0, 0);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
        int t = 0;
        for (; t + D <= half; t += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) { products(d); load(d, t + D + d); }
        }
        // (half a ring is left, or nothing)
        if (t < half)
#pragma unroll
            for (int d = 0; d < D / 2; ++d) products(d);
    }
    float* redb = red + 4 * 9 * 32 * 32;
    bsum += __shfl_xor(bsum, 32, 64);
    if (lhi == 0) redb[wave * 32 + l32] = bsum;
    wgrad_reduce_store<false>(acc, red, a.dW + (size_t)split * a.split_stride, o0, i0, a.cout, a.cin);
    if (i0 == 0 && tid < 32 && o0 + tid < a.cout)
        a.db[(size_t)split * a.split_stride + o0 + tid] = ((redb[tid] + redb[32 + tid]) + redb[64 + tid]) + redb[96 + tid];
}

// Which form a frame's weight gradients take: the float32 instruction where its shorter ends outweigh its longer units, which is where the
// split form's wavefronts have at most two.  us per launch, few / split: 16 x 16 cells, 24 -> 32 -> 24 channels 8.3 / 11.7, 64 channels 7.8 /
// 11.8; 12 x 20, 128 channels 9.8 / 12.4; 16 x 24, 256 -> 128 -> 128 12.2 / 13.5; 24 x 40, 64 channels 10.6 / 12.4 (all two units); 24 x 40, 128
// channels 14.5 / 14.6, 30 x 50, 128 -> 128 -> 64 16.7 / 15.7 (three); 34 x 54, 128 channels 17.4 / 16.5 (four).
WgradForm wgrad_f32_form(const Geo& g)
{
    int s1, s2;
    wgrad_splits_for(g, WGRAD_F32, &s1, &s2);
    const int n_units = cdiv(g.padded_positions(), 16);
    return cdiv(n_units, std::min(s1, s2) * 4) <= 2 ? WGRAD_F32_FEW : WGRAD_F32;
}

static Wgrad32Args wgrad_f32_args(const Plan& p, const float* dY, const float* X, float* dW, float* db, int cin, int cout, int splits)
{
    Wgrad32Args a;
    a.dY = dY; a.X = X; a.dW = dW; a.db = db; a.split_stride = p.grad_stride;
    a.cin = cin; a.cout = cout; a.GX = cdiv(cin, 8); a.GY = cdiv(cout, 8);
    a.PPT = p.PPT; a.guard = p.guard; a.Wp = p.g.Wp;
    a.n_units = cdiv(p.g.padded_positions(), p.wgrad_few ? 8 : 16);
    a.units_per_wave = cdiv(a.n_units, splits * 4);
    a.o_tiles = cdiv(cout, 32); a.i_tiles = cdiv(cin, 32); a.splits = splits;
    a.items_per_xcd = cdiv(a.o_tiles * a.i_tiles * splits, 8);
    return a;
}

// ------------------------------------------------------------------ classifier backward
//   g = d loss / d z from the loss kernel's slots (gather_g), also left in gz;
//   da2[p][o] = [a2[p][o] > 0] * sum_c g[c][p] * W3[c][o];   dW3, db3: one slot per block (the optimiser kernel adds them)
// A block of 512 threads takes 64 padded positions and up to 512 channels (blockIdx.y: which).  Bound by its chain of dependent memory round
// trips, like the bfloat16 kernel of the same layer, and laid out like it: the two products side by side, four wavefronts each, and
// everything that does not depend on g asked for before it is: a2 on its way to LDS, where both products take it from, and the first
// tiles of W3.  256 threads that did one product after the other, each with loads of its own behind g: 68 x 120 cells, 256 -> 128 -> 128 channels
// 673 us a call of four steps, 664 so; 16 x 16 cells, 64 channels 192.7 and 187.0; 90 x 160 cells 1001 and 994, two frames of it 1837 and 1832;
// 135 x 240 cells, 24 -> 32 -> 24 channels 609 and 603.  Wide heads (beyond 256 channels a compute unit has room for one block): 34 x 60 cells,
// 128 -> 128 -> 256 channels 432 and 425, -> 512 599 and 581; 68 x 120, 64 -> 64 -> 512 813 and 796, 32 -> 32 -> 1100 1349 and 1301; 34 x 60, 32 -> 32 -> 1024 669
// and 580.  (Of all this the bands per XCD are 0.1 % of a call, at 90 x 160 cells with 64 channels 1 %.)
constexpr int B32_BP = 64, B32_NT = 512, B32_TILES = 16;
constexpr int B32_RUN = B32_BP * 32 + 160;      // bytes of a run's positions in LDS: 32 of the 64 banks on behind position 31, 40 on from run to
                                                // run, so that the lanes of a dW3 read (four runs, both halves of the positions) have a bank each

template <bool PARTS>       // PARTS: more channels than a block takes
__global__ void __launch_bounds__(B32_NT, 1)
k_conv3_bwd_f32(const float* __restrict__ slots, const float* __restrict__ T, const unsigned long long* __restrict__ n_valid,
                    int CP, LossTiling lt, const float* __restrict__ a2, const float* __restrict__ W3T, float* __restrict__ da2,
                    float* __restrict__ gz, float* __restrict__ part, Geo g, int PPT, int guard, int blocks)
{
    constexpr int BP = B32_BP, GP = BP + 8;     // (pitch: the two halves of a B read 32 banks apart)
    __shared__ __attribute__((aligned(16))) float g_cp[32 * GP];    // [class][position]
    extern __shared__ __attribute__((aligned(16))) unsigned char a2s[];      // [run of eight channels][position][8], see at()
    // (what the first loads need, in one trip for the arguments)
    asm volatile("" ::"s"(slots), "s"(T), "s"(n_valid), "s"(CP), "s"(lt.tiles_x), "s"(lt.tiles_y), "s"(a2), "s"(W3T), "s"(g.n), "s"(g.h), "s"(g.w), "s"(g.Hp), "s"(g.Wp),
                 "s"(g.C), "s"(g.k2), "s"(g.by_frame.d), "s"(g.by_frame.m), "s"(g.by_row.d), "s"(g.by_row.m), "s"(blocks), "s"(PPT), "s"(guard));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int PP = g.padded_positions(), hw = g.h * g.w;
    const int bid = xcd_band(blockIdx.x, blocks), m0 = bid * BP;
    // this block's tiles of 32 channels and runs of eight, from tile t_first on
    const int t_first = PARTS ? blockIdx.y * B32_TILES : 0, OT = (g.c2 + 31) / 32 - t_first, G2 = (g.c2 + 7) / 8 - t_first * 4, CG = (g.C + 7) / 8;
    const int tiles = PARTS ? min(OT, B32_TILES) : OT;
    if (PARTS) { a2 += (size_t)t_first * 4 * PPT * 8; da2 += (size_t)t_first * 4 * PPT * 8; W3T += (size_t)t_first * 4 * 64 * 4; }
    auto at = [](int run, int pos) __attribute__((always_inline)) { return run * B32_RUN + pos * 32 + (pos >= 32 ? 128 : 0); };

    // ---- a2: 16 bytes per thread and turn, 128 of a run's 64 positions; rows behind the last position and runs behind the last one
    //      repeat it
    constexpr int TURNS = 4;                       // turns in registers before the gradient (c2 = 128); the others follow behind it
    const int half = tid & 1, pos = (tid >> 1) & 63, r0 = tid >> 7;
    const size_t col = (size_t)(guard + min(m0 + pos, PP - 1)) * 8 + half * 4;
    f32x4 av[TURNS];
#pragma unroll
    for (int k = 0; k < TURNS; ++k) av[k] = *(const f32x4*)(a2 + (size_t)min(r0 + 4 * k, G2 - 1) * PPT * 8 + col);
    // W3 of the first two tiles that a wavefront of the first product takes (all load them: see the bfloat16 kernel)
    f32x4 wf[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) wf[k][q] = *(const f32x4*)(W3T + ((min((wave & 3) / 2 + 2 * k, tiles - 1) * 4 + q) * 64 + lane) * 4);
    {
        const int pl = tid & 63;
        float v[4];
        const GatherCell cell = gather_g<4, 8>(slots, T, n_valid, CP, lt, g, m0 + pl, PP, wave, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = wave + 8 * k;
            g_cp[c * GP + pl] = c < g.C ? v[k] : 0.f;
            if (c < g.C && cell.inside && t_first == 0) gz[((size_t)cell.img * g.C + c) * hw + cell.cy * g.w + cell.cx] = v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < TURNS; ++k)
        if (r0 + 4 * k < tiles * 4) *(f32x4*)(a2s + at(r0 + 4 * k, pos) + half * 16) = av[k];
    for (int run = r0 + 4 * TURNS; run < tiles * 4; run += 4)
        *(f32x4*)(a2s + at(run, pos) + half * 16) = *(const f32x4*)(a2 + (size_t)min(run, G2 - 1) * PPT * 8 + col);
    __syncthreads();

    float* slot = part + (size_t)bid * (32 * g.k2 + 32);
    if (wave < 4) {
        const int pm = (wave & 1) * 32 + l32, mp = m0 + pm;
        float gb[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) gb[q][e] = g_cp[(q * 8 + lhi * 4 + e) * GP + pm];
        auto tile = [&](int t, const f32x4 (&w)[4]) __attribute__((always_inline)) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < CG)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[q][e], gb[q][e], acc, 0, 0, 0);
            // (g is zero on the border, and so is da2)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t * 4 + q < G2 && mp < PP) {
                    const f32x4 mk = *(const f32x4*)(a2s + at(t * 4 + q, pm) + lhi * 16);
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = mk[e] > 0.f ? acc[q * 4 + e] : 0.f;
                    *(f32x4*)(da2 + ((size_t)(t * 4 + q) * PPT + guard + mp) * 8 + lhi * 4) = v;
                }
        };
        const int t0 = wave >> 1;
        if (t0 < tiles) tile(t0, wf[0]);
        if (t0 + 2 < tiles) tile(t0 + 2, wf[1]);
        for (int t = t0 + 4; t < tiles; t += 2) {
            f32x4 w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = *(const f32x4*)(W3T + ((t * 4 + q) * 64 + lane) * 4);
            tile(t, w);
        }
        // db3: eight threads per class
        const int c = tid >> 3, q = tid & 7;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += g_cp[c * GP + q * 8 + k];
        s += __shfl_xor(s, 1, 64); s += __shfl_xor(s, 2, 64); s += __shfl_xor(s, 4, 64);
        if (q == 0 && c < g.C && t_first == 0) slot[32 * g.k2 + c] = s;
    } else {
        // dW3: k = positions, the two halves of the block's 64
        f32x4 ga[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) ga[q] = *(const f32x4*)(g_cp + l32 * GP + lhi * 32 + q * 4);
        for (int t = wave - 4; t < tiles; t += 4) {
            const float* ab = (const float*)(a2s + at(min((t * 32 + l32) >> 3, G2 - 1), lhi * 32)) + (l32 & 7);
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int s = 0; s < 32; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ga[s >> 2][s & 3], ab[s * 8], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = (r >> 2) * 8 + lhi * 4 + (r & 3);
                const int o = (t_first + t) * 32 + l32;
                if (c < g.C && o < g.k2) slot[c * g.k2 + o] = acc[r];
            }
        }
    }
}

// ------------------------------------------------------------------ host-side entry points
void forward_f32(Ctx& c, const Plan& p, char* ws)
{
    const Geo& g = p.g;
    auto f = [&](size_t at) { return at ? (float*)(ws + at) : nullptr; };
    const float* theta = f(p.theta);
    conv_f32(c, "conv1_fwd_f32", p, 0, f(p.feat), f(p.wq1), theta + p.po.W1, g.c_in, g.c1, f(p.bq1), nullptr, f(p.a1), nullptr, nullptr, nullptr);
    conv_f32(c, "conv2_fwd_logits_f32", p, 2, f(p.a1), f(p.wq2), theta + p.po.W2, g.c1, g.c2, f(p.bq2), nullptr, f(p.a2), f(p.wq3), f(p.zpart), nullptr);
}

void backward_f32(Ctx& c, const Plan& p, char* ws, float* dfeat)
{
    const Geo& g = p.g;
    auto f = [&](size_t at) { return (float*)(ws + at); };
    const int tiles3 = cdiv(g.c2, 32);
    auto classifier = [&](auto kernel) {
        ensure_dynamic_lds((const void*)kernel, (size_t)B32_TILES * 4 * B32_RUN);
        ST_LAUNCH(c, "conv3_bwd_f32", kernel, dim3(p.blocks3, cdiv(tiles3, B32_TILES)), dim3(B32_NT), (size_t)std::min(tiles3, B32_TILES) * 4 * B32_RUN, f(p.g_slots), f(p.tadj),
                  (const unsigned long long*)(ws + p.counters), (g.C + 3) / 4 * 4, p.lt, f(p.a2), f(p.wq3t), f(p.da2), f(p.gz), f(p.grad3), g,
                  p.PPT, p.guard, p.blocks3);
    };
    if (tiles3 <= B32_TILES) classifier(k_conv3_bwd_f32<false>); else classifier(k_conv3_bwd_f32<true>);
    conv_f32(c, "conv2_dgrad_f32", p, 1, f(p.da2), f(p.wq2t), f(p.theta) + p.po.W2, g.c2, g.c1, nullptr, f(p.a1), f(p.da1), nullptr, nullptr, nullptr);
    if (dfeat)
        conv_f32(c, "conv1_dgrad_f32", p, 3, f(p.da1), f(p.wq1t), f(p.theta) + p.po.W1, g.c1, g.c_in, nullptr, nullptr, nullptr, nullptr, nullptr, dfeat);
    float* grad = f(p.grad);
    const Wgrad32Args a1 = wgrad_f32_args(p, f(p.da1), f(p.feat), grad + p.po.W1, grad + p.po.b1, g.c_in, g.c1, p.splits1);
    const Wgrad32Args a2 = wgrad_f32_args(p, f(p.da2), f(p.a1), grad + p.po.W2, grad + p.po.b2, g.c1, g.c2, p.splits2);
    const int blocks1 = a1.items_per_xcd * 8, blocks2 = a2.items_per_xcd * 8;
    const auto kernel = p.wgrad_few ? k_wgrad3x3_f32_few : k_wgrad3x3_f32;
    ensure_dynamic_lds((const void*)kernel, WGRAD_SMEM_BYTES);
    ST_LAUNCH(c, "conv12_wgrad_f32", kernel, dim3(blocks1 + blocks2), dim3(256), WGRAD_SMEM_BYTES, a1, a2, blocks1);
}

}  // namespace st
