// Forward pass of a head without padded buffers: what st_head_forward_noalloc runs where the matrix-core
// kernels' operands -- channels rounded up to 64 or eight, weights in rows of 32, guards of two grid rows --
// do not fit its built-in scratch.  Features and weights are read where the caller has them, and the
// scratch holds the two activations and the logits at their own sizes, nothing else.
//
// The rounding points are those of the other kernels (bfloat16 path: features, weights and activations), the
// sums are float32 and differ from theirs in order only.  A head that ends up here has few channels on a large
// frame (or very many on a tiny one): one thread per cell and four output channels, the
// weights as scalar loads, bound by the cached re-reads of the nine cells under a kernel (with very many
// channels, by the length of that chain).  Whole call, against st_head_forward on padded buffers:
// 810 x 810 cells, 1 -> 1 -> 1 -> 2 125 us (318); 32 frames of 511 x 24, 3 -> 6 -> 3 -> 4 104 us (253);
// 4 x 1 cells, 54 004 -> 2 -> 32 -> 28, 28 to 32 ms (1.05 ms, but 260 MiB of buffers).
#include "st_kernels.hpp"
#include "st_mfma.hpp"

namespace st {

constexpr int DIRECT_O = 4;      // output channels of one thread

template <bool BF16, class T>
__device__ __forceinline__ float operand(T v) { return BF16 ? (float)from_f32<bf16>(to_f32(v)) : to_f32(v); }

// out[img][o][y][x] = relu(b[o] + sum_{i, tap} W[o][i][tap] * X(img, i, y + tap / 3 - 1, x + tap % 3 - 1)), W as the
// caller has it; element (img, i, y, x) of X lies at img * s_img + i * s_ch + y * s_y + x * s_x.
template <bool BF16, class Tin, class Tout>
__global__ void __launch_bounds__(256)
k_direct_conv3x3(const Tin* __restrict__ X, const float* __restrict__ W, const float* __restrict__ b, Tout* __restrict__ out, int n,
                 int h, int w, int cin, int cout, size_t s_img, size_t s_ch, size_t s_y, size_t s_x, int cell_blocks)
{
    const int og = (int)blockIdx.x / cell_blocks, hw = h * w;
    const int cell = ((int)blockIdx.x - og * cell_blocks) * 256 + threadIdx.x;
    if (cell >= n * hw) return;
    const int img = cell / hw, rr = cell - img * hw, y = rr / w, x = rr - y * w;
    size_t at[9];
    bool in[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
        in[t] = yy >= 0 && yy < h && xx >= 0 && xx < w;
        at[t] = img * s_img + (in[t] ? yy * s_y + xx * s_x : y * s_y + x * s_x);      // (off the grid: any element, dropped)
    }
    const float* wo[DIRECT_O];
    float acc[DIRECT_O];
#pragma unroll
    for (int e = 0; e < DIRECT_O; ++e) {
        wo[e] = W + (size_t)min(og * DIRECT_O + e, cout - 1) * cin * 9;
        acc[e] = 0.f;
    }
    for (int i = 0; i < cin; ++i) {
        float v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) v[t] = operand<BF16>(X[at[t] + i * s_ch]);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            v[t] = in[t] ? v[t] : 0.f;
#pragma unroll
            for (int e = 0; e < DIRECT_O; ++e) acc[e] = __builtin_fmaf(operand<BF16>(wo[e][i * 9 + t]), v[t], acc[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < DIRECT_O; ++e) {
        const int o = og * DIRECT_O + e;
        if (o < cout) out[((size_t)img * cout + o) * hw + rr] = from_f32<Tout>(fmaxf(acc[e] + b[o], 0.f));
    }
}

// The logits without their bias, four classes per thread, where the loss kernel looks for its one share:
// [padded position][CP]
template <bool BF16, class E>
__global__ void __launch_bounds__(256)
k_direct_logits(const E* __restrict__ a2, const float* __restrict__ W3, float* __restrict__ parts, Geo g, int CP, int cell_blocks)
{
    const int cg = (int)blockIdx.x / cell_blocks, hw = g.h * g.w;
    const int cell = ((int)blockIdx.x - cg * cell_blocks) * 256 + threadIdx.x;
    if (cell >= g.n * hw) return;
    const int img = cell / hw, rr = cell - img * hw, y = rr / g.w, x = rr - y * g.w;
    const E* src = a2 + (size_t)img * g.c2 * hw + rr;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int o = 0; o < g.c2; ++o) {
        const float v = to_f32(src[(size_t)o * hw]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_fmaf(operand<BF16>(W3[(size_t)min(cg * 4 + e, g.C - 1) * g.c2 + o]), v, acc[e]);
    }
    *(f32x4*)(parts + (((size_t)img * g.Hp + y + 1) * g.Wp + x + 1) * CP + cg * 4) = acc;
}

struct DirectPlan { size_t a1, a2, parts, total; };

static DirectPlan direct_plan(const Geo& g, bool bf16_path)
{
    const size_t cells = (size_t)g.positions(), esz = bf16_path ? 2 : 4;
    auto up = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    DirectPlan d;
    d.a1 = 0;
    d.a2 = d.a1 + up(cells * g.c1 * esz);
    d.parts = d.a2 + up(cells * g.c2 * esz);
    d.total = d.parts + up((size_t)g.padded_positions() * ((g.C + 3) / 4 * 4) * 4);
    return d;
}

size_t direct_forward_bytes(const Geo& g, bool bf16_path) { return direct_plan(g, bf16_path).total; }

template <bool BF16, class Tin, class E>
static void run(Ctx& c, const Geo& g, const Tin* features, const float* params, char* ws)
{
    const DirectPlan d = direct_plan(g, BF16);
    const ParamOffsets po = param_offsets(g);
    E *a1 = (E*)(ws + d.a1), *a2 = (E*)(ws + d.a2);
    float* parts = (float*)(ws + d.parts);
    const int cb = cdiv(g.positions(), 256), CP = (g.C + 3) / 4 * 4;
    const size_t hw = (size_t)g.h * g.w, ci = g.c_in;
    if (g.nhwc)
        ST_LAUNCH(c, "conv1_fwd_direct", (k_direct_conv3x3<BF16, Tin, E>), dim3(cb * cdiv(g.c1, DIRECT_O)), dim3(256), 0, features, params + po.W1,
                  params + po.b1, a1, g.n, g.h, g.w, g.c_in, g.c1, hw * ci, (size_t)1, g.w * ci, ci, cb);
    else
        ST_LAUNCH(c, "conv1_fwd_direct", (k_direct_conv3x3<BF16, Tin, E>), dim3(cb * cdiv(g.c1, DIRECT_O)), dim3(256), 0, features, params + po.W1,
                  params + po.b1, a1, g.n, g.h, g.w, g.c_in, g.c1, hw * ci, hw, (size_t)g.w, (size_t)1, cb);
    ST_LAUNCH(c, "conv2_fwd_direct", (k_direct_conv3x3<BF16, E, E>), dim3(cb * cdiv(g.c2, DIRECT_O)), dim3(256), 0, a1, params + po.W2,
              params + po.b2, a2, g.n, g.h, g.w, g.c1, g.c2, hw * g.c1, hw, (size_t)g.w, (size_t)1, cb);
    ST_LAUNCH(c, "logits_direct", (k_direct_logits<BF16, E>), dim3(cb * (CP / 4)), dim3(256), 0, a2, params + po.W3, parts, g, CP, cb);
}

ZSrc forward_direct(Ctx& c, const Geo& g, bool bf16_path, const void* features, int feat_dtype, const float* params, char* ws, float* z)
{
    if (bf16_path) {
        if (feat_dtype == ST_BF16) run<true, bf16, bf16>(c, g, (const bf16*)features, params, ws);
        else run<true, float, bf16>(c, g, (const float*)features, params, ws);
    } else {
        if (feat_dtype == ST_BF16) run<false, bf16, float>(c, g, (const bf16*)features, params, ws);
        else run<false, float, float>(c, g, (const float*)features, params, ws);
    }
    return ZSrc{(const float*)(ws + direct_plan(g, bf16_path).parts), 1, params + param_offsets(g).b3, z, 0};
}

}  // namespace st
