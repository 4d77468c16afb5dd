// Shared declarations of the partial-distillation library: geometry, workspace plan, launch
// bookkeeping and small device helpers.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/shadowtutor_head.h"

namespace st {

constexpr int UP = 8;  // up-sampling factor of the head's last stage

typedef __bf16 bf16;

// Division by a number the host knows: one high product and a correction (n < 2^31: the quotient of the
// product is at most one short), where the compiler's own division by a variable is some twenty instructions, and a lone
// wavefront issues one in eight cycles or more.
struct FastDiv { unsigned d, m; };
inline FastDiv fast_div(int d) { return FastDiv{(unsigned)d, d == 1 ? 0xFFFFFFFFu : (unsigned)((1ull << 32) / (unsigned)d)}; }
__host__ __device__ __forceinline__ int fast_quot(int n, const FastDiv& f)
{
    const unsigned q = (unsigned)((unsigned long long)(unsigned)n * f.m >> 32);
    return (int)(q + ((unsigned)n - q * f.d >= f.d ? 1u : 0u));
}

// Which of `n` tiles block `block` of n takes: blocks go to the eight XCDs in turn, and every XCD gets a run of consecutive tiles, about the
// same band of rows in every kernel that orders its tiles so.  (The loss kernel and the convolutions deal out runs of ceil(n / 8), whose edges
// lie a few tiles elsewhere; and with a second row of blocks in the grid, n no multiple of eight, that row begins on another XCD.)
__host__ __device__ __forceinline__ int xcd_band(int block, int n)
{
    const int xcd = block & 7, rest = n & 7;
    return (block >> 3) + xcd * (n >> 3) + (xcd < rest ? xcd : rest);
}

// ------------------------------------------------------------------ geometry
// Activations live position-major ("NHWC") on a grid padded by one zero cell on every side, so
// a 3x3 tap is a plain offset and needs no bounds test:
//   element (img, y, x, c)  ->  ((img * Hp + y + 1) * Wp + x + 1) * C + c
// The row pitch Wp is w + 2 rounded up to a multiple of 8 (extra zero columns on the right): a
// step of one row is then a multiple of 16 bytes in the channel-major copies, which keeps the
// weight-gradient kernel's 8-position windows aligned.
struct Geo {
    int n, h, w;     // frames and low-resolution grid
    int Hp, Wp;      // padded grid: h + 2 rows of pitch Wp >= w + 2
    int H, W;        // frame resolution: 8h, 8w
    int c_in, c1, c2, C;
    // Channel pitches of the internal buffers (activations, gradients, operand copies of the weights):
    // c_in, c1, c2 rounded up to what the kernels of the compute path take in one piece.  The channels
    // beyond the caller's count are zero everywhere, and so are the weights that touch them.
    int ki, k1, k2;
    int ignore_index;
    int grouped;     // 1: frame f has a head (parameters, loss, pixel count) of its own
    int nhwc;        // 1: the caller's features are [n, h, w, c_in] instead of [n, c_in, h, w]
    FastDiv by_frame, by_row;    // Hp * Wp; Wp
    bool padded() const { return ki != c_in || k1 != c1 || k2 != c2; }
    __host__ __device__ int heads() const { return grouped ? n : 1; }
    __host__ __device__ int head_of(int img) const { return grouped ? img : 0; }
    __host__ __device__ int positions() const { return n * h * w; }
    __host__ __device__ int padded_positions() const { return n * Hp * Wp; }
    __host__ __device__ long long pixels() const { return (long long)n * H * W; }
};

inline Geo make_geo(const st_head_desc& d)
{
    Geo g;
    g.n = d.n; g.h = d.h; g.w = d.w;
    g.Hp = d.h + 2; g.Wp = (d.w + 2 + 7) / 8 * 8;
    g.H = d.h * UP; g.W = d.w * UP;
    g.c_in = d.c_in; g.c1 = d.c1; g.c2 = d.c2; g.C = d.n_classes;
    // matrix-core kernels: whole 64-channel stages.  (A narrow head costs up to the work of a 64-channel
    // one, but that is matrix-core work on a chip such a head cannot fill anyway: 96 -> 48 -> 48 on
    // 60 x 107 cells went from 3.12 ms per 4-step call on plain kernels to the time of the launches.)
    // float32 kernels: runs of eight channels.
    const int q = d.compute == ST_COMPUTE_BF16 ? 64 : 8;
    g.ki = (d.c_in + q - 1) / q * q; g.k1 = (d.c1 + q - 1) / q * q; g.k2 = (d.c2 + q - 1) / q * q;
    g.ignore_index = d.ignore_index;
    g.grouped = d.grouped ? 1 : 0;
    g.nhwc = d.feat_layout == ST_NHWC ? 1 : 0;
    g.by_frame = fast_div(g.Hp * g.Wp); g.by_row = fast_div(g.Wp);
    return g;
}

// Offsets (in floats) of the six parameter blocks; identical in the caller's flat vector and in
// the internal one.  Only the order *inside* W1 and W2 differs: OIHW outside, [o][kh][kw][i]
// inside (reduction index contiguous for the implicit GEMMs).
struct ParamOffsets {
    size_t W1, b1, W2, b2, W3, b3, total;
};

inline ParamOffsets param_offsets(const Geo& g)
{
    ParamOffsets o;
    o.W1 = 0;
    o.b1 = o.W1 + (size_t)g.c1 * g.c_in * 9;
    o.W2 = o.b1 + g.c1;
    o.b2 = o.W2 + (size_t)g.c2 * g.c1 * 9;
    o.W3 = o.b2 + g.c2;
    o.b3 = o.W3 + (size_t)g.C * g.c2;
    o.total = o.b3 + g.C;
    return o;
}

// ------------------------------------------------------------------ loss-kernel tiling
// The fused up-sample + cross-entropy kernel works on tiles of LOSS_TY x LOSS_TX groups of 8x8
// frame pixels (two threads per pixel column).  A tile touches (LOSS_TY + 2) x (LOSS_TX + 2)
// low-resolution cells and leaves its share of d loss / d z for them in a slot of its own.
constexpr int LOSS_TX = 32;             // 8-pixel column groups per tile
constexpr int LOSS_TY = 1;              // 8-pixel row groups per tile (the kernel and the gather are written for these two)
constexpr int LOSS_CW = LOSS_TX + 2;    // cells per tile row
constexpr int LOSS_CH = LOSS_TY + 2;    // cell rows per tile

struct LossTiling {
    int tiles_x, tiles_y;   // per frame
    __host__ __device__ int tiles() const { return tiles_x * tiles_y; }
};

inline LossTiling loss_tiling(const Geo& g)
{
    LossTiling t;
    t.tiles_x = (g.w + LOSS_TX - 1) / LOSS_TX;
    t.tiles_y = (g.h + LOSS_TY - 1) / LOSS_TY;
    return t;
}

// ------------------------------------------------------------------ workspace plan
struct Plan {
    Geo g;
    ParamOffsets po;
    LossTiling lt;
    bool bf16;          // compute path
    size_t esz;         // bytes per activation element
    // With several heads (Geo::grouped) every per-head buffer holds heads() consecutive blocks:
    // theta, vel, vel2, best (head_stride floats apart), grad (grad_copies * grad_stride floats
    // apart), grad3 (blocks3 slots apart), the bfloat16 weight copies (their own size apart),
    // the pixel counters (one each).
    int splits1, splits2;   // position splits (per head) of the layer-1 / layer-2 weight-gradient kernels
    bool wgrad_few;         // float32 path: those kernels by the float32 instruction
    int blocks3;            // per-block partial slots (per head) of the layer-3 backward kernel
    int grad_copies;        // max of the splits: partial gradient copies the update sums
    size_t grad_stride;     // floats between two copies (total rounded up to 128 bytes; plans of a forward pass: 16)
    size_t head_stride;     // floats between two heads' parameters (the same)
    int guard;          // guard rows before and after every position-major activation buffer;
                        // also the number of guard columns in front of a channel-major row
    int PPT;            // row pitch (elements) of the channel-major copies; columns per run of channels (float32)
    // byte offsets (activations: of position 0; float32: of the first guard column of the first run)
    size_t feat, a1, a2, da1, da2;
    size_t featT, a1T, da1T, da2T;        // channel-major copies [C][PPT] for the weight-gradient kernels
    size_t grad3;                         // per-block partials of dW3 / db3
    size_t z, g_slots, gz, tadj;   // gz: float32 path (elsewhere room that nothing uses); tadj: U^T of the one-hot labels, [n, C, h, w] float32
    size_t lab8;                   // the labels as bytes, [n, 8h, 8w]: the class, or 255 for a pixel that does not count
    size_t zpart; int z_parts;     // shares of the logits left by the classifier-fused convolution, one per 64 channels (float32: 32)
    size_t theta, vel, vel2, grad, best;   // vel: velocity or Adam's m; vel2: Adam's v
    size_t wq1, wq1t, wq2, wq2t, wq3;      // operand copies of the weights: bfloat16, or float32 in its kernels' order
    size_t bq1, bq2;                       // biases followed by zeros, where the kernels read beyond the counts
    size_t wq3t;                           // W3 transposed, [k2][32 classes] (zero beyond C): MFMA A fragments of its backward
    size_t loss_part, counters, label_counts, conf, scal;   // label_counts: per label block of the opening launch
    size_t bytes_w1, bytes_w1t, bytes_w2, bytes_w2t, bytes_w3, bytes_w3t;   // sizes of the operand copies
    size_t total;
};

// PLAN_FORWARD: room for the buffers of the full plan, with the offsets of those that only training needs set to 0
// (absent), so that no kernel fills them; heads and partial gradients 16 bytes apart.  PLAN_COMPACT: the same buffers without room for
// the others.
enum PlanKind { PLAN_FULL, PLAN_FORWARD, PLAN_COMPACT };
Plan make_plan(const st_head_desc& d, PlanKind kind = PLAN_FULL);

// ------------------------------------------------------------------ launch bookkeeping
// Each kernel launch goes through Launch: it records the kernel's name for the optional event
// profile and turns a launch failure into ST_ERR_HIP instead of an abort.
struct Ctx {
    hipStream_t stream;
    int status;   // first failure sticks
    bool no_profile = false;   // launches of this call never carry profile events
};

// When the event profile is on and covers `name`, hands out a start/stop event pair that the
// launch attaches to the dispatch itself (hipExtLaunchKernelGGL): the pair then times the kernel
// only and puts no extra packet into the stream.  Otherwise both come back null.
void prof_events(Ctx& c, const char* name, hipEvent_t* start, hipEvent_t* stop);
void set_hip_error(hipError_t e);
void ensure_dynamic_lds(const void* kernel, size_t bytes);

#define ST_LAUNCH(ctx, name, kernel, grid, block, shmem, ...)                                   \
    do {                                                                                        \
        if ((ctx).status == ST_OK) {                                                            \
            hipEvent_t e0_ = nullptr, e1_ = nullptr;                                            \
            st::prof_events((ctx), name, &e0_, &e1_);                                           \
            if (e0_)                                                                            \
                hipExtLaunchKernelGGL(kernel, grid, block, shmem, (ctx).stream, e0_, e1_, 0,    \
                                      __VA_ARGS__);                                             \
            else                                                                                \
                hipLaunchKernelGGL(kernel, grid, block, shmem, (ctx).stream, __VA_ARGS__);      \
            hipError_t err_ = hipGetLastError();                                                \
            if (err_ != hipSuccess) { st::set_hip_error(err_); (ctx).status = ST_ERR_HIP; }     \
        }                                                                                       \
    } while (0)

// ------------------------------------------------------------------ device helpers
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
template <class E> __device__ __forceinline__ E from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }  // RNE

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

}  // namespace st
