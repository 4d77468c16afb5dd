// Optimiser step over the flat parameter buffer (fused with the sum of the partial weight
// gradients and the bfloat16 operand copies of the new weights), the per-step bookkeeping
// kernel (loss, per-frame mean IoU) and the stand-alone confusion-matrix / mean-IoU kernels.
#include <string.h>

#include <algorithm>

#include "st_kernels.hpp"
#include "st_mfma.hpp"
#include "st_begin.hpp"
#include "st_finish.hpp"

namespace st {

// One kernel closes a training step; its blocks play three roles (block index ranges):
//
//  (1) optimiser step over the parameters in front of the classifier: theta <- theta - lr * v,
//      v <- mu * v + g (mu == 0: v is not touched), or an Adam step (Section 5.2 of the paper;
//      AdamStep).  g is the sum, in ascending order, of the partial gradients the weight-gradient
//      kernel left behind: `splits1` copies for W1/b1, `splits2` for W2/b2 (its position splits,
//      `stride` floats apart).
//  (2) the same for W3/b3, of which the classifier's backward kernel left one slot per block: L3_RUNS (8)
//      threads per parameter, each adding a contiguous run of the slots, then the runs in order.
//  (3) bookkeeping of the forward pass that preceded the step: block f: mean IoU of frame f from
//      its confusion counts (copied out when asked, then cleared for the next pass); one more
//      block: the tile losses added in a fixed order (float64) over the number of valid pixels.
//
// Roles (1) and (2) also refresh the operand copies of the new weights:
//   wq1, wq2, wq3 : for the forward convolutions; bq1, bq2: their biases, where padded channels follow
//   wq2t          : W2 with the roles of o and i exchanged and the taps mirrored (tap' = 8 - tap),
//                   for the data-gradient of layer 2 run as a forward convolution
//   wq1t          : the same for W1, only when the caller wants the gradient of the features
//   wq3t          : W3 transposed, for the classifier's backward kernel
// bfloat16 path: wq1, wq2, wq2t in fragment order (wfrag_index), wq3 [class][k2], wq3t [k2][32] with
// zero columns beyond the classes.  Float32 path (F32): wq1, wq2, wq2t in fragment order, times F32_SPLIT_SCALE where the layer
// runs on split operands (conv_f32_weight_scale), wq3t in the order of wfrag32_index, wq3 [32][c2 rounded up to 32].  Rows and columns of padded channels and
// classes are cleared by the launch that opens the call and never written later.
struct UpdateArgs {
    float* theta; float* vel; float* vel2; float* grad; size_t stride; int splits1, splits2;
    void *wq1, *wq1t, *wq2, *wq2t, *wq3, *wq3t; float* bq1; float* bq2;   // (bf16 or float elements)
    ParamOffsets po; int c_in, c1, c2, ki, k1, k2;   // k: channel pitches of the operand copies
    float scale1, scale1t, scale2, scale2t;   // float32 path: factors of wq1, wq1t, wq2, wq2t
    float lr, mu;
    int adam; AdamStep ad;   // adam != 0: vel = first moment m, vel2 = second moment v
    // the launch that opens a call: the caller's vectors (its OIHW order) from which theta and, where there are any, the
    // optimiser's state vectors are taken
    const float *ext_in, *ext_vel, *ext_vel2;
    // role (2)
    const float* part3; int blocks3; size_t slot3; int C;
    // block ranges; vec: role (1) handles four parameters per thread over [0, W3).  (When a call opens, the blocks behind
    // nb_main handle [W3, total) one by one.)
    int nb_main, nb_l3, nb_finish, vec;
    // role (1) by tiles of 32 x 32 weights under one tap (tiled_block): blocks of W1 and of W2, input-channel tiles of either
    int tiled, nb_t1, nb_t2; FastDiv by_it1, by_it2;
    // several heads (blockIdx.y): floats / elements from one head's block to the next in the
    // parameter-like vectors (theta, vel, vel2), the caller's vectors, the partial gradients,
    // the bfloat16 copies and the layer-3 slots
    size_t hs_param, hs_ext, hs_grad, hs_wq1, hs_wq2, hs_wq3, hs_part3;
    // early-exit form only: receives theta as it was before the step (theta's order), or null
    float* save_old;
};


// Where an internal parameter index j ([o][kh][kw][i]) of a 3x3 block lies.  (A head has fewer than
// 2^30 parameters: 32-bit divisions, a 64-bit one is some forty instructions longer.)
struct Weight3x3 { unsigned o, tap, i; };
__device__ __forceinline__ Weight3x3 weight3x3(unsigned r, unsigned cin)
{
    const unsigned row = r / cin, o = row / 9u;
    return Weight3x3{o, row - o * 9u, r - row * cin};
}

constexpr int PAD_PER_THREAD = 4;     // runs of the padding role per thread

// index in the caller's vector (3x3 weights OIHW) of the internal parameter j ([o][kh][kw][i])
__device__ __forceinline__ unsigned external_index(const UpdateArgs& a, unsigned j)
{
    if (j < (unsigned)a.po.b1) {
        const Weight3x3 k = weight3x3(j, a.c_in);
        return (k.o * a.c_in + k.i) * 9u + k.tap;
    }
    const unsigned w2 = (unsigned)a.po.W2;
    if (j >= w2 && j < (unsigned)a.po.b2) {
        const Weight3x3 k = weight3x3(j - w2, a.c1);
        return w2 + (k.o * a.c1 + k.i) * 9u + k.tap;
    }
    return j;
}

// the operand copies of W1 (layer 1) or W2 for the parameter (o, tap, i) and, with N == 4, the three behind
// it along i
template <bool F32, int N>
__device__ __forceinline__ void copy_weights(const UpdateArgs& a, int layer, const Weight3x3& k, const float (&w)[N])
{
    void* fwd = layer == 1 ? a.wq1 : a.wq2;
    void* bwd = layer == 1 ? a.wq1t : a.wq2t;
    const int kin = layer == 1 ? a.ki : a.k1, kout = layer == 1 ? a.k1 : a.k2;
    if (F32) {
        const float s = layer == 1 ? a.scale1 : a.scale2, st = layer == 1 ? a.scale1t : a.scale2t;
        float* f = (float*)fwd + wfrag_index(k.o, k.tap, k.i, kin);
        if (N == 4) *(f32x4*)f = f32x4{w[0] * s, w[N > 1 ? 1 : 0] * s, w[N > 2 ? 2 : 0] * s, w[N > 3 ? 3 : 0] * s};
        else f[0] = w[0] * s;
        if (bwd)
#pragma unroll
            for (int e = 0; e < N; ++e) ((float*)bwd)[wfrag_index(k.i + e, 8 - k.tap, k.o, kout)] = w[e] * st;
    } else {
        bf16* f = (bf16*)fwd + wfrag_index(k.o, k.tap, k.i, kin);
        bf16 q[N];
#pragma unroll
        for (int e = 0; e < N; ++e) q[e] = (bf16)w[e];
        if (N == 4) *(bf16x4*)f = bf16x4{q[0], q[N > 1 ? 1 : 0], q[N > 2 ? 2 : 0], q[N > 3 ? 3 : 0]};
        else f[0] = q[0];
        if (bwd)
#pragma unroll
            for (int e = 0; e < N; ++e) ((bf16*)bwd)[wfrag_index(k.i + e, 8 - k.tap, k.o, kout)] = q[e];
    }
}

// What an update reads besides the gradient: the parameters and the optimiser's state, one or four of each.  Asked for before the
// gradient's partial copies (or the classifier's slots) are, so that both are one trip to memory: the optimiser launch is a
// chain of such trips.  90 x 160 cells: 6.8 -> 6.4 us a launch; 16 x 16 cells, seven copies, in two trips instead of five: a call 192.5 -> 191.3.
template <class V> struct Held { V w, m, v; };
template <class V>
__device__ __forceinline__ Held<V> held(const UpdateArgs& a, unsigned j)
{
    Held<V> h = {};
    h.w = *(const V*)(a.theta + j);
    if (a.adam || a.mu != 0.f) h.m = *(const V*)(a.vel + j);
    if (a.adam) h.v = *(const V*)(a.vel2 + j);
    return h;
}

// (EE: the early-exit form's extras -- save_old here, the host copy of the metric in finish_block --
//  are compiled in; the kernels of the fixed-step form never look at those fields)
template <bool EE, bool F32, bool OPEN>
__device__ __forceinline__ void apply_update(const UpdateArgs& a, unsigned j, float g, const Held<float>& h)
{
    float w;
    if (OPEN) {
        const unsigned x = external_index(a, j);
        w = a.ext_in[x];
        if (a.ext_vel) a.vel[j] = a.ext_vel[x];
        if (a.ext_vel2) a.vel2[j] = a.ext_vel2[x];
        a.theta[j] = w;
    } else {
        w = h.w;
        if (EE && a.save_old) a.save_old[j] = w;
        if (a.adam) {
            const float m = __builtin_fmaf(a.ad.beta1, h.m, a.ad.one_minus_beta1 * g);
            const float v = __builtin_fmaf(a.ad.beta2, h.v, a.ad.one_minus_beta2 * (g * g));
            a.vel[j] = m;
            a.vel2[j] = v;
            w = w - a.ad.step_scale * m / (__fsqrt_rn(v) * a.ad.inv_sqrt_bc2 + a.ad.eps);
        } else {
            if (a.mu != 0.f) {
                const float v = __builtin_fmaf(a.mu, h.m, g);
                a.vel[j] = v;
                g = v;
            }
            w = __builtin_fmaf(-a.lr, g, w);
        }
        a.theta[j] = w;
    }
    if (j < a.po.b1) {
        copy_weights<F32>(a, 1, weight3x3(j, a.c_in), {w});
    } else if (j < a.po.W2) {
        if (a.bq1) a.bq1[j - a.po.b1] = w;
    } else if (j < a.po.b2) {
        copy_weights<F32>(a, 2, weight3x3(j - (unsigned)a.po.W2, a.c1), {w});
    } else if (j < a.po.W3) {
        if (a.bq2) a.bq2[j - a.po.b2] = w;
    } else if (j < a.po.b3) {
        const unsigned r = j - (unsigned)a.po.W3;
        const unsigned cl = r / (unsigned)a.c2, o = r - cl * a.c2;
        if (OPEN && a.wq3t && (int)cl == a.C - 1) {
            // the call opens: the classes beyond the last are zeros (nothing writes them later)
            for (unsigned k = cl + 1; k < 32; ++k) {
                if (F32) ((float*)a.wq3t)[wfrag32_index(o, k, 32)] = 0.f;
                else ((bf16*)a.wq3t)[o * 32 + k] = (bf16)0.f;
            }
        }
        if (F32) {
            ((float*)a.wq3)[cl * ((a.c2 + 31) & ~31) + o] = w;
            if (a.wq3t) ((float*)a.wq3t)[wfrag32_index(o, cl, 32)] = w;
        } else {
            ((bf16*)a.wq3)[cl * a.k2 + o] = (bf16)w;
            if (a.wq3t) ((bf16*)a.wq3t)[o * 32 + cl] = (bf16)w;
        }
    }
}

// One step of four consecutive parameters; their new values.
template <bool EE>
__device__ __forceinline__ f32x4 step4(const UpdateArgs& a, unsigned j, f32x4 g, const Held<f32x4>& h)
{
    f32x4 w = h.w;
    if (EE && a.save_old) *(f32x4*)(a.save_old + j) = w;
    if (a.adam) {
        f32x4 m, v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            m[e] = __builtin_fmaf(a.ad.beta1, h.m[e], a.ad.one_minus_beta1 * g[e]);
            v[e] = __builtin_fmaf(a.ad.beta2, h.v[e], a.ad.one_minus_beta2 * (g[e] * g[e]));
            w[e] = w[e] - a.ad.step_scale * m[e] / (__fsqrt_rn(v[e]) * a.ad.inv_sqrt_bc2 + a.ad.eps);
        }
        *(f32x4*)(a.vel + j) = m;
        *(f32x4*)(a.vel2 + j) = v;
    } else {
        if (a.mu != 0.f) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(a.mu, h.m[e], g[e]);
            *(f32x4*)(a.vel + j) = v;
            g = v;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = __builtin_fmaf(-a.lr, g[e], w[e]);
    }
    *(f32x4*)(a.theta + j) = w;
    return w;
}

// Four consecutive parameters (all block boundaries below W3 are multiples of four here, and so are
// the channel counts: the four lie in the same block and under the same tap).
template <bool EE, bool F32, bool OPEN>
__device__ __forceinline__ void apply_update4(const UpdateArgs& a, unsigned j, f32x4 g, const Held<f32x4>& h)
{
    f32x4 w;
    if (OPEN) {
        unsigned x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[e] = external_index(a, j + e); w[e] = a.ext_in[x[e]]; }
        if (a.ext_vel) *(f32x4*)(a.vel + j) = f32x4{a.ext_vel[x[0]], a.ext_vel[x[1]], a.ext_vel[x[2]], a.ext_vel[x[3]]};
        if (a.ext_vel2) *(f32x4*)(a.vel2 + j) = f32x4{a.ext_vel2[x[0]], a.ext_vel2[x[1]], a.ext_vel2[x[2]], a.ext_vel2[x[3]]};
        *(f32x4*)(a.theta + j) = w;
    } else {
        w = step4<EE>(a, j, g, h);
    }
    if (j < a.po.b1) copy_weights<F32>(a, 1, weight3x3(j, a.c_in), {w[0], w[1], w[2], w[3]});
    else if (j < a.po.W2) {
        if (a.bq1) *(f32x4*)(a.bq1 + (j - a.po.b1)) = w;
    } else if (j < a.po.b2) copy_weights<F32>(a, 2, weight3x3(j - (unsigned)a.po.W2, a.c1), {w[0], w[1], w[2], w[3]});
    else if (a.bq2) *(f32x4*)(a.bq2 + (j - a.po.b2)) = w;
}

// acc + the partial gradients s0 .. s0 + N - 1 of `splits`, in ascending order (s0 == 0: their sum); N loads in flight, those beyond the
// last copy repeat it and are not added.
template <int N, class V>
__device__ __forceinline__ V add_copies(V acc, const float* gp, size_t stride, int s0, int splits)
{
    V v[N];
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = *(const V*)(gp + (size_t)min(s0 + e, splits - 1) * stride);
#pragma unroll
    for (int e = 0; e < N; ++e)
        if (s0 + e < splits) acc = s0 + e ? acc + v[e] : v[e];
    return acc;
}
// Loads that only repeat the last copy are left out for the counts of large layers and many clients, two to five, where a launch is bound by
// its bytes: two copies of 3.5 million parameters 18.67 us with three loads, 18.47 with two, three or four of 1.3 million, five loads each,
// 0.1 % of a 16-step call.  Six copies and more are small layers, bound by the trip, and a form for each count costs more in
// branches than it saves: 16 copies 6.5 -> 6.7 us, 8 copies 6.8 -> 7.1, 5 copies of 0.44 million 6.0 -> 6.25 (one alone: two loads, in the noise).
template <class V>
__device__ __forceinline__ V sum_copies(const float* gp, size_t stride, int splits)
{
    V g = {};
    if (splits <= 2) return add_copies<2>(g, gp, stride, 0, splits);
    if (splits == 3) return add_copies<3>(g, gp, stride, 0, splits);
    if (splits == 4) return add_copies<4>(g, gp, stride, 0, splits);
    if (splits == 5) return add_copies<5>(g, gp, stride, 0, splits);
    for (int s = 0; s < splits; s += 8) g = add_copies<8>(g, gp, stride, s, splits);
    return g;
}

// Role (1) on tiles (bfloat16 path, channel counts that are multiples of 32): a block takes 32 output x 32 input channels of a 3x3
// layer under one tap, four input channels per thread.  A wavefront then has eight output channels' 128 bytes of every vector, and
// leaves whole lines of both operand copies: the forward one as it is (in the order of wfrag_index eight output channels' eight
// inputs are 128 bytes), the mirrored one, whose runs go over eight output channels, through LDS.  By consecutive parameters the
// forward copy goes out in pieces of 16 bytes, each line's in eight wavefronts of as many XCDs, and the mirrored one in pieces of
// two.  Bound by those lines' way to memory: 256 -> 256 -> 256 channels 10.8 -> 7.5 us a launch.
template <bool EE>
__device__ __forceinline__ void tiled_block(const UpdateArgs& a, int b)
{
    __shared__ __attribute__((aligned(16))) bf16 turn[256 * 4];
    const int tid = threadIdx.x;
    if (b >= a.nb_t1 + a.nb_t2) {
        // the biases, one by one
        const unsigned x = (unsigned)(b - a.nb_t1 - a.nb_t2) * 256 + tid;
        if (x >= (unsigned)(a.c1 + a.c2)) return;
        const unsigned j = x < (unsigned)a.c1 ? (unsigned)a.po.b1 + x : (unsigned)a.po.b2 + (x - a.c1);
        const Held<float> h = held<float>(a, j);
        apply_update<EE, false, false>(a, j, sum_copies<float>(a.grad + j, a.stride, x < (unsigned)a.c1 ? a.splits1 : a.splits2), h);
        return;
    }
    const bool one = b < a.nb_t1;
    const FastDiv by_it = {one ? a.by_it1.d : a.by_it2.d, one ? a.by_it1.m : a.by_it2.m};
    const int t = one ? b : b - a.nb_t1, q = fast_quot(t, by_it), it = t - q * (int)by_it.d, ot = q / 9, tap = q - ot * 9;
    const int ci = one ? a.c_in : a.c1, o = ot * 32 + (tid >> 3), i = it * 32 + (tid & 7) * 4;
    const unsigned j = (one ? 0u : (unsigned)a.po.W2) + (unsigned)((o * 9 + tap) * ci + i);
    const Held<f32x4> h = held<f32x4>(a, j);
    const f32x4 w = step4<EE>(a, j, sum_copies<f32x4>(a.grad + j, a.stride, one ? a.splits1 : a.splits2), h);
    const bf16x4 v = {(bf16)w[0], (bf16)w[1], (bf16)w[2], (bf16)w[3]};
    *(bf16x4*)((bf16*)(one ? a.wq1 : a.wq2) + wfrag_index(o, tap, i, one ? a.ki : a.k1)) = v;
    bf16* const bwd = (bf16*)(one ? a.wq1t : a.wq2t);
    if (!bwd) return;
    // (a wavefront's own 32 inputs x 8 outputs: no other touches them.  Its lanes read what others of them wrote, LDS serves a wavefront in
    //  order: what lies between keeps the compiler to that order and is no instruction)
    bf16* const mine = turn + (tid >> 6) * 256;
#pragma unroll
    for (int e = 0; e < 4; ++e) mine[((tid & 7) * 4 + e) * 8 + ((tid >> 3) & 7)] = v[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int lane = tid & 63;
    if (lane < 32)
        *(bf16x8*)(bwd + wfrag_index(it * 32 + lane, 8 - tap, ot * 32 + (tid >> 6) * 8, one ? a.k1 : a.k2)) = *(const bf16x8*)(mine + lane * 8);
}

// Classifier's role of k_step_end: values per block, and the runs its threads split the slots into.
constexpr int L3_VALUES = 32, L3_RUNS = 256 / L3_VALUES;

// acc + the sum of src[s * stride] over s0 <= s < s1; N loads in flight.  Loads beyond the end repeat the last
// slot (`n` slots) and are not added.  The N values are added in pairs, pairs of pairs, ..: one after the other, 966 slots in eight
// runs are 2.05e-7 of their 2-norm off (and in 16 runs 1.6e-7), so 0.95e-7, at the same time.
template <int N>
__device__ __forceinline__ float add_slots(float acc, const float* src, size_t stride, int s0, int s1, int n)
{
    float v[N];
    src += (size_t)s0 * stride;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        v[e] = *src;
        src += s0 + e + 1 < n ? stride : 0;
    }
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = s0 + e < s1 ? v[e] : 0.f;
#pragma unroll
    for (int k = 1; k < N; k *= 2)
#pragma unroll
        for (int e = 0; e < N; e += 2 * k) v[e] += v[e + k];
    return acc + v[0];
}

// (OPEN: as a role of the launch that opens a call: parameters in, operand copies; no other roles, so that the
//  launch carries none of their LDS.  TILED: role (1) by tiles, a kernel of its own because two kilobytes more of LDS and the
//  longer code cost the launch that has no tiles 0.1 us)
template <bool EE, bool F32, bool OPEN, bool TILED = false>
__device__ __forceinline__ void step_end_block(UpdateArgs a, const FinishArgs& f, int b, int head)
{
    if (head) {
        if (a.theta) { a.theta += head * a.hs_param; a.vel += head * a.hs_param; a.vel2 += head * a.hs_param; }
        if (EE && a.save_old) a.save_old += head * a.hs_param;
        if (a.grad) a.grad += head * a.hs_grad;
        // (several heads: bfloat16 path only)
        auto move = [](void*& q, size_t by) { if (q) q = (bf16*)q + by; };
        move(a.wq1, head * a.hs_wq1); move(a.wq1t, head * a.hs_wq1);
        move(a.wq2, head * a.hs_wq2); move(a.wq2t, head * a.hs_wq2);
        move(a.wq3, head * a.hs_wq3); move(a.wq3t, head * (size_t)a.k2 * 32);
        if (a.ext_in) a.ext_in += head * a.hs_ext;
        if (a.ext_vel) a.ext_vel += head * a.hs_ext;
        if (a.ext_vel2) a.ext_vel2 += head * a.hs_ext;
        if (a.part3) a.part3 += head * a.hs_part3;
    }
    if (b < a.nb_main) {
        if constexpr (TILED) { tiled_block<EE>(a, b); return; }
        // role (1), four parameters per thread over [0, W3): the partial gradients are added in
        // ascending order of the split, up to eight in flight
        if (a.vec) {
            const unsigned j = ((unsigned)b * 256 + threadIdx.x) * 4;
            if (j >= a.po.W3) return;
            Held<f32x4> h = {};
            f32x4 g = {0.f, 0.f, 0.f, 0.f};
            if (!OPEN) {
                h = held<f32x4>(a, j);
                g = sum_copies<f32x4>(a.grad + j, a.stride, j < a.po.W2 ? a.splits1 : a.splits2);
            }
            apply_update4<EE, F32, OPEN>(a, j, g, h);
            return;
        }
        // role (1), one parameter per thread
        const unsigned j = (unsigned)b * 256 + threadIdx.x;
        if (j >= a.po.W3) return;
        Held<float> h = {};
        float g = 0.f;
        if (!OPEN) {
            h = held<float>(a, j);
            g = sum_copies<float>(a.grad + j, a.stride, j < a.po.W2 ? a.splits1 : a.splits2);
        }
        apply_update<EE, F32, OPEN>(a, j, g, h);
    } else if constexpr (OPEN) {
        // [W3, total) one by one
        const unsigned j = (unsigned)a.po.W3 + (unsigned)(b - a.nb_main) * 256 + threadIdx.x;
        if (j < a.po.total) apply_update<EE, F32, OPEN>(a, j, 0.f, Held<float>{});
    } else if (b < a.nb_main + a.nb_l3) {
        // role (2): slot layout [32 classes][k2] weights, then [32] biases.  The slots were
        // written by other compute units, so every load is a round trip to memory: the role is
        // laid out for few of them, and for whole 128-byte lines.  A block takes 32 consecutive values; its 256 threads
        // split the slots into 8 contiguous runs (thread = value + 32 * run), every thread adds its
        // run group by group (add_slots), and the 8 partial sums of a value are added in the order of the runs.  A run of up to 32
        // slots is one trip; a longer one is added 16 at a time, because then the slots' bytes bind and more loads in
        // flight only get in the way of the parameters' (966 slots of 256 channels, 21 MB: the launch takes 18.6 us with 16,
        // 20.9 with 32, 21.4 with 24).  16 values in 16 runs of 8 loads fetched every line twice and made two trips where
        // this makes one: 242 slots of 128 channels (90 x 160 cells) 7.1 -> 6.3 us, four heads of those 14.9 -> 14.1,
        // 516 slots (135 x 240 cells) 8.2 -> 8.2, the 966 slots 20.2 -> 18.6.  64 values in 4 runs: 7.2 us at 242 slots, 24.3 at 966.
        __shared__ float run_sum[L3_RUNS][L3_VALUES];
        const int kk = threadIdx.x % L3_VALUES, run = threadIdx.x / L3_VALUES;
        const int k = (b - a.nb_main) * L3_VALUES + kk;
        const int n_w = a.C * a.c2;
        const bool live = k < n_w + a.C;
        Held<float> h = {};
        if (run == 0 && live) h = held<float>(a, (unsigned)a.po.W3 + k);
        float acc = 0.f;
        if (live) {
            const float* src = a.part3 + (k < n_w ? (size_t)(k / a.c2) * a.k2 + k % a.c2 : (size_t)32 * a.k2 + (k - n_w));
            const int per = (a.blocks3 + L3_RUNS - 1) / L3_RUNS;
            const int s1 = min((run + 1) * per, a.blocks3);
            int s = run * per;
            for (; s1 - s > 32; s += 16) acc = add_slots<16>(acc, src, a.slot3, s, s1, a.blocks3);
            if (s1 - s > 16) acc = add_slots<32>(acc, src, a.slot3, s, s1, a.blocks3);
            else if (s1 - s > 8) acc = add_slots<16>(acc, src, a.slot3, s, s1, a.blocks3);
            else if (s1 > s) acc = add_slots<8>(acc, src, a.slot3, s, s1, a.blocks3);
        }
        run_sum[run][kk] = acc;
        __syncthreads();
        if (run == 0 && live) {
            float total = run_sum[0][kk];
#pragma unroll
            for (int r = 1; r < L3_RUNS; ++r) total += run_sum[r][kk];
            if (F32) a.grad[a.po.W3 + k] = total;      // (the float32 path's gradient can be looked at as a whole)
            apply_update<EE, F32, OPEN>(a, (unsigned)a.po.W3 + k, total, h);
        }
    } else finish_block<EE>(f, b - a.nb_main - a.nb_l3, head);
}

template <bool EE, bool F32, bool TILED = false>
__global__ void __launch_bounds__(256) k_step_end(UpdateArgs a, FinishArgs f)
{
    step_end_block<EE, F32, false, TILED>(a, f, blockIdx.x, blockIdx.y);
}

// Bookkeeping of a pass without an update and, behind it, what the call hands back: nb_out blocks per vector -- theta,
// then the optimiser's state -- to the caller's order.
// (Optimiser state once took a launch per vector and direction: four of 5.2 us in an Adam call at 90 x 160 cells,
//  256 -> 128 -> 128 channels.  Riding here and on the opening launch they cost 3 us together: such a call 728 -> 710 us, one with momentum at
//  135 x 240 cells 1268 -> 1251.)
// A thread takes a parameter of the caller's order, so that whole lines are written and the scattered side is reads (a block's 256 are
// nine rows of 28, which the caches hold).  The other way round every line was written in nine parts (10.9 MiB counted at 256 -> 128 -> 128
// channels, 8.5 now): the launch 8.0 us and now 7.0 at 135 x 240 cells with momentum, 9.6 and now 8.7 with Adam's two moments at 90 x 160.
struct HandBack {
    int nb_finish, nb_out;
    const float* src[3]; float* dst[3];
    ParamOffsets po; FastDiv by_in1, by_in2;      // (channels of a row of W1, of W2)
    size_t hs_param, hs_ext;     // several heads: floats from one head's vector to the next
};

template <bool EE>
__global__ void __launch_bounds__(256) k_finish_pass(HandBack a, FinishArgs f)
{
    if ((int)blockIdx.x < a.nb_finish) {
        finish_block<EE>(f, blockIdx.x, blockIdx.y);
        return;
    }
    const int b = blockIdx.x - a.nb_finish, v = b / a.nb_out;
    const unsigned x = (unsigned)(b - v * a.nb_out) * 256 + threadIdx.x;
    const float* src = (v == 0 ? a.src[0] : v == 1 ? a.src[1] : a.src[2]) + blockIdx.y * a.hs_param;
    float* dst = (v == 0 ? a.dst[0] : v == 1 ? a.dst[1] : a.dst[2]) + blockIdx.y * a.hs_ext;
    if (x < a.po.total) dst[x] = src[internal_index(a.po, a.by_in1, a.by_in2, x)];
}

// Zeros for the padding of the operand copies: channels beyond the caller's counts, of which the parameter role writes
// nothing (so the two roles share a launch: 64-channel stages of 48 channels in front of 60 x 107 cells once had a clearing
// launch of their own, 4 us of a 270 us call).  A thread takes runs of the four 3x3 copies, in the order they are
// stored -- a run is one row's and tap's next eight k -- and then the small ones' rests.
template <bool F32>
__device__ __forceinline__ void pad_block(const UpdateArgs& a, unsigned block, unsigned n_runs)
{
    constexpr int W = 8, R32 = 32, B = W * (F32 ? 4 : 2);
    const int c[3] = {a.c_in, a.c1, a.c2}, k[3] = {a.ki, a.k1, a.k2};
    auto rows = [&](int m) { return F32 ? (k[m] + R32 - 1) / R32 * R32 : k[m]; };
    void* const copy[4] = {a.wq1, a.wq2, a.wq1t, a.wq2t};
    const int row_of[4] = {1, 2, 0, 1}, k_of[4] = {0, 1, 1, 2};
#pragma unroll 1
    for (int u = 0; u < PAD_PER_THREAD; ++u) {
        unsigned i = (block * PAD_PER_THREAD + u) * 256 + threadIdx.x;
        if (i < n_runs) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                if (!copy[m]) continue;
                const int K = k[k_of[m]], rv = c[row_of[m]], kv = c[k_of[m]];
                const unsigned runs = (unsigned)rows(row_of[m]) * 9u * (unsigned)(K / W);
                if (i >= runs) { i -= runs; continue; }
                const unsigned t = i >> 5, per = (unsigned)K / W;
                const int row = (int)(t / per / 9u * 32u + (i & 31)), k0 = (int)(t % per) * W;
                char* dst = (char*)copy[m] + (size_t)i * B;
                if (row >= rv || k0 >= kv) {
#pragma unroll
                    for (int e = 0; e < B; e += 16) *(u32x4*)(dst + e) = u32x4{0u, 0u, 0u, 0u};
                } else if (k0 + W > kv)
                    for (int e = kv - k0; e < W; ++e) { if (F32) ((float*)dst)[e] = 0.f; else ((bf16*)dst)[e] = (bf16)0.f; }
                break;
            }
        } else {
            // per channel of the second layer behind its last one: its column of wq3, its row of wq3t; biases
            i -= n_runs;
            const unsigned rest2 = (unsigned)(rows(2) - a.c2), kr1 = (unsigned)((a.k1 + R32 - 1) / R32 * R32), kr2 = (unsigned)((a.k2 + R32 - 1) / R32 * R32);
            if (i < rest2 * 32) {
                const int o = a.c2 + (int)(i >> 5), cl = (int)(i & 31);
                if (F32) {
                    if (cl < a.C) ((float*)a.wq3)[cl * rows(2) + o] = 0.f;
                    if (a.wq3t) ((float*)a.wq3t)[wfrag32_index(o, cl, 32)] = 0.f;
                } else {
                    if (cl < a.C) ((bf16*)a.wq3)[cl * a.k2 + o] = (bf16)0.f;
                    if (a.wq3t) ((bf16*)a.wq3t)[o * 32 + cl] = (bf16)0.f;
                }
                continue;
            }
            i -= rest2 * 32;
            if (i < kr1 - a.c1) { a.bq1[a.c1 + i] = 0.f; continue; }
            i -= kr1 - a.c1;
            if (i < kr2 - a.c2) a.bq2[a.c2 + i] = 0.f;
        }
    }
}

// the runs of eight k of a head's 3x3 operand copies, and the blocks of pad_block (none without padding)
static unsigned pad_runs(const Plan& p, const UpdateArgs& a)
{
    return (unsigned)(((a.wq1 ? p.bytes_w1 : 0) + (a.wq2 ? p.bytes_w2 : 0) + (a.wq1t ? p.bytes_w1t : 0) + (a.wq2t ? p.bytes_w2t : 0)) / (8 * p.esz));
}
static int pad_blocks(const Plan& p, const UpdateArgs& a)
{
    const Geo& g = p.g;
    // (float32 path: rows rounded up to 32)
    if (!g.padded() && (p.bf16 || (g.c_in % 32 == 0 && g.c1 % 32 == 0 && g.c2 % 32 == 0))) return 0;
    const auto r32 = [](int k) { return (k + 31) / 32 * 32; };
    const long long rest = 32ll * ((p.bf16 ? g.k2 : r32(g.k2)) - g.c2) + (r32(g.k1) - g.c1) + (r32(g.k2) - g.c2);
    return cdiv(pad_runs(p, a) + rest, 256 * PAD_PER_THREAD);
}

// The launch that opens a call: kinds of blocks that do not depend on each other,
//   first   U^T of the label map and the pixel counts (label_adjoint_block),
//   then    the caller's parameters into theta and the operand copies: the blocks of
//           k_step_end, head by head,
//   then    zeros for the padding of the operand copies (pad_block), where channels are padded,
//   then    feature packing (pack_features_block),
//   last    clearing what later kernels expect to be zero (ZeroList).
// Run one after the other they are four short launches, each of which leaves most of the chip
// idle for most of its time.
struct BeginArgs {
    const void* features; void* feat; void* featT; int in_bf16, PPT, guard;
    int pack_vec;                          // the 16-byte packing role
    int pack_x, pack_y, nb_pack;           // pack grid: pack_x position (16-byte role: column) tiles x pack_y channel tiles (x rows)
    const int32_t* labels; const uint8_t* wmap; float* T; unsigned int* counts; int CP, nb_label;
    uint8_t* lab8;                         // the labels as bytes for the loss kernel (written by the label role)
    int nb_update, nb_update_all;          // blocks of the parameter role per head, and of all heads
    int nb_pad; unsigned pad_runs;         // blocks and runs of the padding role (one head: heads of their own are not padded)
    Geo g;
};

template <bool F32>
__global__ void __launch_bounds__(256) k_call_begin(BeginArgs q, UpdateArgs a, ZeroList z)
{
    extern __shared__ __attribute__((aligned(16))) float dyn_lds[];
    int b = blockIdx.x;
    // (blocks start in index order: the label blocks, each a long chain of dependent steps, go
    //  first, the short packing blocks last)
    if (b < q.nb_label) {
        float* colsum = dyn_lds;
        unsigned int* cnt_part = (unsigned int*)(dyn_lds + q.CP * LABEL_PITCH);
        label_adjoint_block(q.labels, q.wmap, q.T, q.counts + b, q.g, b, colsum, cnt_part, q.CP, q.lab8);
        return;
    }
    b -= q.nb_label;
    if (b >= q.nb_update_all) {
        b -= q.nb_update_all;
        if (b < q.nb_pad) { pad_block<F32>(a, (unsigned)b, q.pad_runs); return; }
        b -= q.nb_pad;
        if (b >= q.nb_pack) { zero_block(z, b - q.nb_pack); return; }
        const int bx = b % q.pack_x, by = (b / q.pack_x) % q.pack_y, bz = b / (q.pack_x * q.pack_y);
        if (F32) {
            if (q.in_bf16) pack_features_f32_block((const bf16*)q.features, (float*)q.feat, q.g, q.PPT, q.guard, bx, by);
            else pack_features_f32_block((const float*)q.features, (float*)q.feat, q.g, q.PPT, q.guard, bx, by);
            return;
        }
        if (q.pack_vec) {
            pack_features_vec_block((const bf16*)q.features, (bf16*)q.feat, (bf16*)q.featT, q.g, q.PPT, q.guard, bx, by, bz, (bf16*)dyn_lds);
            return;
        }
        if (q.in_bf16) pack_features_block((const bf16*)q.features, (bf16*)q.feat, (bf16*)q.featT, q.g, q.PPT, q.guard, bx, by, (bf16*)dyn_lds);
        else pack_features_block((const float*)q.features, (bf16*)q.feat, (bf16*)q.featT, q.g, q.PPT, q.guard, bx, by, (bf16*)dyn_lds);
        return;
    }
    step_end_block<false, F32, true>(a, FinishArgs{}, b % q.nb_update, b / q.nb_update);
}

FinishArgs finish_args(const Plan& p, char* ws, float* loss_out, double* miou_out, long long* conf_out,
                       double* miou_host, unsigned long long* token_host, unsigned long long token)
{
    FinishArgs f;
    f.loss_part = (const float*)(ws + p.loss_part);
    f.n_part = loss_blocks(p.g);
    f.n_valid = (const unsigned long long*)(ws + p.counters);
    f.conf = (unsigned long long*)(ws + p.conf);
    f.n = p.g.n; f.C = p.g.C;
    f.fph = p.g.n / p.g.heads();
    f.pph = f.n_part / p.g.heads();
    f.loss_out = loss_out;
    f.miou_a = (double*)(ws + p.scal);   // per-frame metric kept in the workspace (host-side loop exits)
    f.miou_b = miou_out;                 // the caller's array (may be null)
    f.miou_c = miou_host;                // host memory the device can write (may be null): the loop exits read it
    f.token_c = token_host; f.token = token;
    f.conf_out = conf_out;
    return f;
}

static void head_strides(UpdateArgs& a, const Plan& p)
{
    a.hs_param = p.head_stride;
    a.hs_ext = p.po.total;
    a.hs_grad = p.grad_stride * p.grad_copies;
    a.hs_wq1 = (size_t)p.g.k1 * 9 * p.g.ki;
    a.hs_wq2 = (size_t)p.g.k2 * 9 * p.g.k1;
    a.hs_wq3 = (size_t)p.g.C * p.g.k2;
    a.hs_part3 = (size_t)p.blocks3 * conv3_bwd_slot_floats(p.g);
}

// do_step: optimiser step (else, when a call opens: theta from ext_in and the operand copies);
// finish: also close the forward pass that preceded it (loss, per-frame mIoU, counts)
static int step_end_args(const Plan& p, char* ws, float lr, float mu, const AdamStep* adam, bool do_step, bool finish,
                         const float* ext_in, bool w1t, const FinishArgs& f, UpdateArgs& a, float* save_old = nullptr)
{
    a.theta = (float*)(ws + p.theta);
    a.save_old = do_step ? save_old : nullptr;
    a.vel = (float*)(ws + p.vel);
    a.vel2 = (float*)(ws + p.vel2);
    a.ext_in = do_step ? nullptr : ext_in; a.ext_vel = a.ext_vel2 = nullptr;
    a.adam = adam ? 1 : 0;
    if (adam) a.ad = *adam; else memset(&a.ad, 0, sizeof(a.ad));
    a.grad = (float*)(ws + p.grad);
    a.stride = p.grad_stride;
    a.splits1 = p.splits1;
    a.splits2 = p.splits2;
    auto at = [&](size_t off) -> void* { return off ? ws + off : nullptr; };
    a.wq1 = at(p.wq1); a.wq1t = w1t ? at(p.wq1t) : nullptr;
    a.wq2 = at(p.wq2); a.wq2t = at(p.wq2t);
    a.wq3 = at(p.wq3); a.wq3t = at(p.wq3t);
    a.bq1 = (float*)at(p.bq1); a.bq2 = (float*)at(p.bq2);
    a.po = p.po; a.c_in = p.g.c_in; a.c1 = p.g.c1; a.c2 = p.g.c2; a.ki = p.g.ki; a.k1 = p.g.k1; a.k2 = p.g.k2;
    const Geo& g = p.g;
    a.scale1 = conv_f32_weight_scale(g, g.c_in, g.c1); a.scale1t = conv_f32_weight_scale(g, g.c1, g.c_in);
    a.scale2 = conv_f32_weight_scale(g, g.c1, g.c2); a.scale2t = conv_f32_weight_scale(g, g.c2, g.c1);
    a.lr = lr; a.mu = mu;
    a.part3 = (const float*)(ws + p.grad3);
    a.blocks3 = p.blocks3; a.slot3 = conv3_bwd_slot_floats(p.g); a.C = p.g.C;
    // four parameters per thread when every block below W3, and every row under one tap, starts at a
    // multiple of four
    a.vec = (p.g.c_in % 4 == 0 && p.g.c1 % 4 == 0 && p.g.c2 % 4 == 0) ? 1 : 0;
    a.nb_main = a.vec ? cdiv(p.po.W3 / 4, 256) : cdiv(p.po.W3, 256);
    a.nb_t1 = p.g.c1 / 32 * 9 * (p.g.c_in / 32); a.nb_t2 = p.g.c2 / 32 * 9 * (p.g.c1 / 32);
    a.by_it1 = fast_div(std::max(p.g.c_in / 32, 1)); a.by_it2 = fast_div(std::max(p.g.c1 / 32, 1));
    // Tiles where one head has one or more to each of the 256 CUs: there they always pay.  The launch at 720p, medians in us by consecutive
    // parameters -> by tiles, SGD unless noted: 360 tiles 5.9 -> 5.7 (momentum 6.6 -> 6.2; four heads of 360, the whole call 1534 -> 1495), 432
    // 8.2 -> 7.1, 504 6.0 -> 5.7.  (Larger heads were measured before partial gradients began with whole lines, which both ways gained by: 576
    // 8.2 -> 7.0, 864 6.7 -> 6.5 with 320, 256 and 64 channels and 8.0 -> 6.6 with 192, 256 and 128, Adam 9.2 -> 8.6; 1008 10.4 -> 7.1, 1152
    // 10.8 -> 7.5, Adam 12.9 -> 10.0; 1296 11.9 -> 9.6, momentum 13.2 -> 11.0, four frames 19.35 -> 16.2.)  Below the line they are level for one
    // head of few tiles and worth 1 to 2 % of a call from some 130 on, or of heads that have as many together; the line does not follow that.
    // Calls of four steps at 16 x 24 / 45 x 80 / 90 x 160 cells: 18 tiles 146.3 -> 147.1 / 173.3 -> 173.4 / 256.9 -> 255.3, 72 149.2 -> 148.5 /
    // 177.6 -> 176.4 / 261.5 -> 260.3, 108 153.7 -> 153.9 / 184.1 -> 183.8 / 267.8 -> 267.3, 135 161.3 -> 160.3 / 200.8 -> 199.3 / 290.2 -> 288.0, 162
    // 162.3 -> 160.2 / 204.5 -> 202.2 / 296.6 -> 294.2, 225 169.1 -> 165.8 / 210.5 -> 208.1 / 353.6 -> 351.7; 315 175.5 -> 171.2 / 219.4 -> 216.8 /
    // 378.7 -> 378.0; eight heads of 72 166.5 -> 160.6 / 346.5 -> 338.5 / 751 -> 746.
    a.tiled = do_step && p.bf16 && p.g.c_in % 32 == 0 && p.g.c1 % 32 == 0 && p.g.c2 % 32 == 0 && a.nb_t1 + a.nb_t2 >= 256;
    if (a.tiled) a.nb_main = a.nb_t1 + a.nb_t2 + cdiv(p.g.c1 + p.g.c2, 256);
    const int nb_tail = do_step ? 0 : cdiv(p.po.total - p.po.W3, 256);
    a.nb_l3 = do_step ? cdiv(p.g.C * p.g.c2 + p.g.C, L3_VALUES) : 0;
    a.nb_finish = finish ? f.fph + 1 : 0;
    head_strides(a, p);
    return a.nb_main + nb_tail + a.nb_l3 + a.nb_finish;
}

void step_end(Ctx& c, const Plan& p, char* ws, float lr, float mu, const AdamStep* adam, bool finish, float* loss_out,
              double* miou_out, long long* conf_out, bool w1t, float* save_old)
{
    UpdateArgs a;
    const FinishArgs f = finish_args(p, ws, loss_out, miou_out, conf_out);
    const int blocks = step_end_args(p, ws, lr, mu, adam, true, finish, nullptr, w1t, f, a, save_old);
    const char* name = adam ? (finish ? "adam_update+finish_pass" : "adam_update") : (finish ? "sgd_update+finish_pass" : "sgd_update");
    auto go = [&](auto kernel) { ST_LAUNCH(c, name, kernel, dim3(blocks, p.g.heads()), dim3(256), 0, a, f); };
    if (a.tiled) { if (a.save_old) go(k_step_end<true, false, true>); else go(k_step_end<false, false, true>); }
    else if (p.bf16) { if (a.save_old) go(k_step_end<true, false>); else go(k_step_end<false, false>); }
    else { if (a.save_old) go(k_step_end<true, true>); else go(k_step_end<false, true>); }
}

// Whether the packing role can move 16 bytes at a time: bfloat16 path, bfloat16 features whose rows are
// multiples of 16 bytes from a 16-byte aligned start, in the [n, c_in, h, w] order, no padded channels.
static bool pack_vectors(const Plan& p, const void* features, int feat_dtype)
{
    return p.bf16 && !p.g.nhwc && feat_dtype == ST_BF16 && p.g.w % 8 == 0 && !p.g.padded() && ((uintptr_t)features & 15) == 0;
}

// Opens a call in one launch: packs the features, takes the caller's parameters (OIHW order)
// into theta and the operand copies and, where there are any, the optimiser's `state` vectors, clears `zero` and, with labels, computes T = U^T (one-hot valid
// labels) and every label block's pixel count (the first loss pass adds them up).
void call_begin(Ctx& c, const Plan& p, char* ws, const void* features, int feat_dtype, const float* head_params,
                bool w1t, const int32_t* labels, const uint8_t* wmap, const ZeroList& zero, const float* vel, const float* vel2)
{
    const Geo& g = p.g;
    BeginArgs q;
    memset(&q, 0, sizeof(q));
    q.features = features; q.feat = ws + p.feat;
    q.featT = p.featT ? ws + p.featT : nullptr;
    q.in_bf16 = feat_dtype == ST_BF16;
    q.PPT = p.PPT; q.guard = p.guard;
    q.pack_vec = pack_vectors(p, features, feat_dtype) ? 1 : 0;
    if (!p.bf16) {
        q.pack_x = cdiv(g.padded_positions(), 256); q.pack_y = g.ki / 8;
        q.nb_pack = q.pack_x * q.pack_y;
    } else if (q.pack_vec) {
        q.pack_x = cdiv(g.Wp, 64); q.pack_y = g.c_in / 64;
        q.nb_pack = q.pack_x * q.pack_y * g.n * g.Hp;
    } else {
        q.pack_x = cdiv(g.padded_positions(), 64); q.pack_y = g.ki / 64;
        q.nb_pack = q.pack_x * q.pack_y;
    }
    q.g = g;
    q.CP = (g.C + 3) / 4 * 4;
    if (labels) {
        q.labels = labels; q.wmap = wmap; q.T = (float*)(ws + p.tadj); q.lab8 = (uint8_t*)(ws + p.lab8);
        q.counts = (unsigned int*)(ws + p.label_counts);
        q.nb_label = label_blocks(g);
    }
    UpdateArgs a;
    const FinishArgs f = finish_args(p, ws, nullptr, nullptr, nullptr);
    q.nb_update = step_end_args(p, ws, 0.f, 0.f, nullptr, false, false, head_params, w1t, f, a);
    a.ext_vel = vel; a.ext_vel2 = vel2;
    q.nb_update_all = q.nb_update * g.heads();
    q.nb_pad = pad_blocks(p, a); q.pad_runs = pad_runs(p, a);
    if (zero.overflow) { c.status = ST_ERR_SHAPE; return; }
    size_t lds = p.bf16 ? (size_t)64 * PACKV_PITCH * sizeof(bf16) : 0;
    if (labels) lds = std::max(lds, (size_t)(q.CP * LABEL_PITCH + 4) * sizeof(float));
    const int nb_zero = zero.n ? zero.first[zero.n] : 0;
    auto go = [&](auto kernel) {
        ST_LAUNCH(c, labels ? "pack+label_adjoint+params_in" : "pack+params_in", kernel,
                  dim3(q.nb_label + q.nb_update_all + q.nb_pad + q.nb_pack + nb_zero), dim3(256), lds, q, a, zero);
    };
    if (p.bf16) go(k_call_begin<false>); else go(k_call_begin<true>);
}

int label_blocks(const Geo& g) { return g.n * g.h * cdiv(g.w, LABEL_TX); }

// bookkeeping of a pass without an update; with ext_out the same launch hands theta (and with out_vel, out_vel2 the
// optimiser's state) back to the caller's vectors (OIHW order), none of which may overlap
void finish_pass(Ctx& c, const Plan& p, char* ws, float* loss_out, double* miou_out, long long* conf_out,
                 float* ext_out, double* miou_host, unsigned long long* token_host, unsigned long long token,
                 float* out_vel, float* out_vel2)
{
    const FinishArgs f = finish_args(p, ws, loss_out, miou_out, conf_out, miou_host, token_host, token);
    HandBack a;
    memset(&a, 0, sizeof(a));
    a.nb_finish = f.fph + 1;
    int vectors = 0;
    if (ext_out) {
        a.nb_out = cdiv(p.po.total, 256);
        a.po = p.po; a.by_in1 = fast_div(p.g.c_in); a.by_in2 = fast_div(p.g.c1);
        a.hs_param = p.head_stride; a.hs_ext = p.po.total;
        const size_t from[3] = {p.theta, p.vel, p.vel2};
        float* const to[3] = {ext_out, out_vel, out_vel2};
        for (; vectors < 3 && to[vectors]; ++vectors) { a.src[vectors] = (const float*)(ws + from[vectors]); a.dst[vectors] = to[vectors]; }
    }
    const dim3 grid(a.nb_finish + vectors * a.nb_out, p.g.heads());
    const char* name = ext_out ? "finish_pass+params_out" : "finish_pass";
    if (miou_host) ST_LAUNCH(c, name, k_finish_pass<true>, grid, dim3(256), 0, a, f);
    else ST_LAUNCH(c, name, k_finish_pass<false>, grid, dim3(256), 0, a, f);
}

// ------------------------------------------------------------------ stand-alone metric
// Confusion counts of a class map against labels.  Each block keeps its own C x C table in
// LDS and adds it to the result at the end; integer counts, so the order of additions does
// not matter.  Few, large blocks: the final additions of every block land on the same few
// cache lines.  Per trip a wavefront takes 1024 consecutive pixels as four label loads of 16
// bytes and four prediction loads of 4 bytes per lane, each instruction reading one contiguous
// stretch, all issued before the first is used.  Label maps are piecewise constant, so most
// wavefronts hold a single (label, prediction) pair: that case is detected with one ballot and
// costs one LDS addition.  Otherwise every lane merges equal neighbours among its 16 pixels
// and adds each run to the table itself; LDS resolves lanes that hit the same counter.  (Counting the
// pairs of the stretch's two ends with ballots and adding only other pixels one by one: 12.7 us at 1920 x 1080
// with 2 % of the pixels off, against 7.6 -- most pixel slots of a wavefront then hold one of those.)
// Tables too large for LDS (more than 128 classes) go to the result directly, one addition
// per distinct pair of a wavefront and pixel slot.
// (Blocks of 512 threads, one per compute unit at 1920 x 1080 instead of half as many: 8.2 against 7.6 us, the
// merge has twice the additions.  The last block in computing the mean IoU instead of a launch of its own:
// 18.2 us for this kernel -- additions that must complete before a block counts itself in, and a table
// read back past the caches -- against 7.6 + 3.7.)
constexpr int CONF_THREADS = 1024;
constexpr int CONF_PER_T = 16;                       // pixels of one thread per trip
constexpr int CONF_MAX_BLOCKS = 256;
constexpr int MIOU_THREADS = 1024;

// Mean IoU (Eq. 1) of a C x C table of counts, any C up to 256: 16 lanes per class add
// that class's row and column (exact integer sums), then a single thread adds the per-class
// ratios of the classes that occur as a label in ascending order in float64 (eight read at a time: read one by one they are a
// chain of LDS latencies) and divides by their number; 0 when there is none.  A table of up to 64 classes is fetched once, by all threads, into LDS.
__global__ void __launch_bounds__(MIOU_THREADS)
k_miou_from_counts(const unsigned long long* __restrict__ conf, int C, double* __restrict__ out)
{
    __shared__ unsigned long long tab[64 * 64];
    __shared__ double iou[256];
    __shared__ int present[256];
    const bool staged = C <= 64;
    if (staged) {
        for (int i = threadIdx.x; i < C * C; i += MIOU_THREADS) tab[i] = conf[i];
        __syncthreads();
    }
    const int sub = threadIdx.x & 15;
    for (int c = threadIdx.x >> 4; c < (C + 3) / 4 * 4; c += MIOU_THREADS / 16) {      // (whole wavefronts)
        unsigned long long row = 0, col = 0;
        if (c < C)
            for (int k = sub; k < C; k += 16) {
                row += staged ? tab[c * C + k] : conf[c * C + k];
                col += staged ? tab[k * C + c] : conf[k * C + c];
            }
#pragma unroll
        for (int d = 8; d; d >>= 1) { row += __shfl_xor(row, d, 64); col += __shfl_xor(col, d, 64); }
        if (sub == 0 && c < C) {
            const unsigned long long inter = staged ? tab[c * C + c] : conf[c * C + c];
            present[c] = row != 0;
            iou[c] = row ? (double)inter / (double)(row + col - inter) : 0.0;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        int cnt = 0;
        for (int c0 = 0; c0 < C; c0 += 8) {
            double t[8];
            int p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { t[e] = iou[min(c0 + e, C - 1)]; p[e] = present[min(c0 + e, C - 1)]; }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (c0 + e < C) { sum += t[e]; cnt += p[e]; }      // (a class that does not occur adds zero)
        }
        *out = cnt ? sum / cnt : 0.0;
    }
}

template <bool LDS_TABLE>
__global__ void __launch_bounds__(CONF_THREADS)
k_confusion(const uint8_t* __restrict__ pred, const int32_t* __restrict__ labels, long long P, int C,
            int ignore, unsigned long long* __restrict__ conf)
{
    extern __shared__ unsigned int table[];
    if (LDS_TABLE) {
        for (int i = threadIdx.x; i < C * C; i += CONF_THREADS) table[i] = 0;
        __syncthreads();
    }
    const bool aligned = (((uintptr_t)labels | (uintptr_t)pred) & 15) == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long trip = (long long)CONF_THREADS * CONF_PER_T;
    for (long long first = (long long)blockIdx.x * trip; first < P; first += (long long)gridDim.x * trip) {
        // pixel (k, j) of this lane: wbase + 256 k + 4 lane + j
        const long long wbase = first + (long long)wave * (64 * CONF_PER_T);
        if (wbase >= P) continue;
        int bins[CONF_PER_T];
        if (aligned && wbase + 64 * CONF_PER_T <= P) {
            u32x4 lv[4];
            unsigned int pv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) lv[k] = *(const u32x4*)(labels + wbase + 256 * k + 4 * lane);
#pragma unroll
            for (int k = 0; k < 4; ++k) pv[k] = *(const unsigned int*)(pred + wbase + 256 * k + 4 * lane);
#pragma unroll
            for (int i = 0; i < CONF_PER_T; ++i) {
                const int y = (int)lv[i >> 2][i & 3];
                const int q = (int)((pv[i >> 2] >> (8 * (i & 3))) & 0xFFu);
                bins[i] = ((unsigned)y < (unsigned)C && q < C) ? y * C + q : -1;
            }
            if ((unsigned)ignore < (unsigned)C) {        // (an ignored label that is also a class index)
#pragma unroll
                for (int i = 0; i < CONF_PER_T; ++i)
                    if ((int)lv[i >> 2][i & 3] == ignore) bins[i] = -1;
            }
        } else {
#pragma unroll
            for (int i = 0; i < CONF_PER_T; ++i) {
                const long long at = wbase + 256 * (i >> 2) + 4 * lane + (i & 3);
                bins[i] = -1;
                if (at < P) {
                    const int y = labels[at];
                    const int q = pred[at];
                    if (y != ignore && y >= 0 && y < C && q < C) bins[i] = y * C + q;
                }
            }
        }
        if (LDS_TABLE) {
            const int b0 = __builtin_amdgcn_readfirstlane(bins[0]);
            bool same = true;
#pragma unroll
            for (int i = 0; i < CONF_PER_T; ++i) same &= bins[i] == b0;
            if (__ballot(same) == __ballot(true)) {
                // one pair for the whole wavefront (or nothing to count)
                if (b0 >= 0 && lane == 0) atomicAdd(&table[b0], 64u * CONF_PER_T);
            } else {
                unsigned int run = 1;
#pragma unroll
                for (int i = 1; i <= CONF_PER_T; ++i) {
                    if (i < CONF_PER_T && bins[i] == bins[i - 1]) { ++run; continue; }
                    if (bins[i - 1] >= 0) atomicAdd(&table[bins[i - 1]], run);
                    run = 1;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < CONF_PER_T; ++i) {
                const int bin = bins[i];
                unsigned long long todo = __ballot(bin >= 0);
                while (todo) {
                    const int leader = __ffsll((long long)todo) - 1;
                    const int lbin = __shfl(bin, leader, 64);
                    const unsigned long long same = __ballot(bin == lbin);
                    if (lane == leader) atomicAdd(&conf[lbin], (unsigned long long)__popcll(same));
                    todo &= ~same;
                }
            }
        }
    }
    if (LDS_TABLE) {
        __syncthreads();
        for (int i = threadIdx.x; i < C * C; i += CONF_THREADS)
            if (table[i]) atomicAdd(&conf[i], (unsigned long long)table[i]);
    }
}

__global__ void __launch_bounds__(256) k_clear_counts(unsigned long long* conf, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) conf[i] = 0ull;
}

void confusion_and_miou(Ctx& c, const uint8_t* pred, const int32_t* labels, long long P, int C, int ignore,
                        long long* conf, double* miou)
{
    ST_LAUNCH(c, "zero_fill", k_clear_counts, dim3(cdiv(C * C, 256)), dim3(256), 0, (unsigned long long*)conf, C * C);
    const int blocks = std::min(std::max(cdiv(P, CONF_THREADS * CONF_PER_T), 1), CONF_MAX_BLOCKS);
    const size_t lds = (size_t)C * C * 4;
    if (lds <= 64 * 1024)
        ST_LAUNCH(c, "confusion", (k_confusion<true>), dim3(blocks), dim3(CONF_THREADS), lds, pred, labels, P, C, ignore,
                  (unsigned long long*)conf);
    else
        ST_LAUNCH(c, "confusion", (k_confusion<false>), dim3(blocks), dim3(CONF_THREADS), 0, pred, labels, P, C, ignore,
                  (unsigned long long*)conf);
    ST_LAUNCH(c, "miou", k_miou_from_counts, dim3(1), dim3(MIOU_THREADS), 0, (const unsigned long long*)conf, C, miou);
}

}  // namespace st
