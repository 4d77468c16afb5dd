// Host-side launchers of the kernels, one group per source file.
#pragma once
#include "st_common.hpp"

namespace st {

struct FinishArgs;   // st_finish.hpp: arguments of the bookkeeping role

// k_layout.hip
// regions to clear, each 16-byte aligned and padded to 16 bytes (`count` of them, `stride` bytes apart);
// a role of the launch that opens a call clears them all
struct ZeroList {
    static constexpr int MAX = 24;
    char* ptr[MAX]; size_t stride[MAX]; unsigned n16[MAX]; int first[MAX + 1], per[MAX]; int n = 0; bool overflow = false;
    ZeroList() { first[0] = 0; }
    void add(void* p, size_t bytes, int count = 1, size_t stride_bytes = 0);
};
// Region r owns blocks [first[r], first[r + 1]), per[r] of them for each of its repetitions, each block
// (256 threads) a fixed run of ZERO_PER_BLOCK 16-byte words.
constexpr int ZERO_PER_BLOCK = 256 * 8;
__device__ __forceinline__ void zero_block(const ZeroList& z, int block)
{
    int r = 0;
    while (r + 1 < z.n && block >= z.first[r + 1]) ++r;     // block-uniform, n is small
    const int local = block - z.first[r], rep = local / z.per[r];
    uint4* p = (uint4*)(z.ptr[r] + (size_t)rep * z.stride[r]);
    const unsigned base = (unsigned)(local - rep * z.per[r]) * ZERO_PER_BLOCK;
#pragma unroll
    for (int k = 0; k < ZERO_PER_BLOCK / 256; ++k) {
        const unsigned i = base + (unsigned)k * 256 + threadIdx.x;
        if (i < z.n16[r]) p[i] = make_uint4(0, 0, 0, 0);
    }
}
// Where the parameter x of the caller's vector lies in the internal one (by_in1, by_in2: c_in and c1 as divisors): inside a 3x3 weight block
//   internal (o*9 + tap)*ci + i   <->   external (o*ci + i)*9 + tap.
__device__ __forceinline__ unsigned internal_index(const ParamOffsets& po, FastDiv by_in1, FastDiv by_in2, unsigned x)
{
    const bool one = x < (unsigned)po.b1;
    if (!one && !(x >= (unsigned)po.W2 && x < (unsigned)po.b2)) return x;
    const unsigned base = one ? 0u : (unsigned)po.W2;
    // (Chosen word by word: chosen as a whole it went through scratch memory, and the launch that closes a call took that much longer:
    //  key frame at 90 x 160 cells 547.2 -> 545.5 us and 587.9 -> 583.2 on two cards, with Adam's state 556.7 -> 552.7 and 600.5 -> 592.5)
    const FastDiv by_in = {one ? by_in1.d : by_in2.d, one ? by_in1.m : by_in2.m};
    const unsigned oi = (x - base) / 9u, tap = x - base - oi * 9u;
    const unsigned o = (unsigned)fast_quot((int)oi, by_in), i = oi - o * by_in.d;
    return base + (o * 9u + tap) * by_in.d + i;
}
void permute_params(Ctx& c, const Plan& p, const float* src, float* dst);

// what the weight gradients of the 3x3 layers run on (float32: split operands, or the float32 instruction)
enum WgradForm { WGRAD_BF16, WGRAD_F32, WGRAD_F32_FEW };

// k_conv_f32.hip -- the float32 path's kernels
// factor of the copy of the weights that a 3x3 layer of cin -> cout channels reads
float conv_f32_weight_scale(const Geo& g, int cin, int cout);
WgradForm wgrad_f32_form(const Geo& g);
void forward_f32(Ctx& c, const Plan& p, char* ws);
void backward_f32(Ctx& c, const Plan& p, char* ws, float* dfeat);

// k_conv_mfma.hip, k_wgrad_mfma.hip, k_conv3_mfma.hip -- matrix-core kernels of the bfloat16 path
void conv3x3_mfma(Ctx& c, const char* name, const Plan& p, const bf16* X, const bf16* Wq, const float* bias,
                  const bf16* mask, bf16* Y, bf16* YT, int cin, int cout, int epi,
                  const bf16* W3q = nullptr, float* zpart = nullptr, float* dense = nullptr);
void wgrad_splits_for(const Geo& g, WgradForm form, int* splits1, int* splits2);
void wgrad3x3_mfma(Ctx& c, const Plan& p, const bf16* da1T, const bf16* featT, const bf16* da2T,
                   const bf16* a1T, float* grad);
int conv3_bwd_blocks(const Geo& g);
size_t conv3_bwd_slot_floats(const Geo& g);
// finish: the bookkeeping of the pass that precedes this backward pass rides on the launch (a few more blocks)
void conv3_bwd_mfma(Ctx& c, const Plan& p, const float* slots, const float* T,
                    const unsigned long long* n_valid, const bf16* a2, const bf16* W3T,
                    bf16* da2, bf16* da2T, float* part,
                    const FinishArgs* finish = nullptr);

// k_loss.hip
size_t loss_slot_floats(const Geo& g);
int loss_blocks(const Geo& g);
// The low-resolution logits as the classifier-fused convolution left them: shares
// [n_parts][padded position][classes rounded up to a multiple of four], added in ascending order
// together with the bias b3; the kernel also writes the sums to the planar tensor z_out
// [n, C, h, w] (each tile its own cells).
struct ZSrc {
    const float* parts; int n_parts; const float* b3; float* z_out;
    size_t b3_stride;     // floats between the biases of two heads (one head per frame)
};
// One more block per head adds up the label blocks' pixel counts (the first pass of a call: the kernels that divide
// by the number of valid pixels come behind it).
struct CountSum { const unsigned int* counts; int per_head; unsigned long long* n_valid; };

// k_head_direct.hip -- forward pass on buffers of the head's own sizes (one head only): the logits for
// loss_pass.  `ws` holds direct_forward_bytes; z: the planar tensor to leave, or null
size_t direct_forward_bytes(const Geo& g, bool bf16_path);
ZSrc forward_direct(Ctx& c, const Geo& g, bool bf16_path, const void* features, int feat_dtype, const float* params, char* ws, float* z);

// labels8: the labels as bytes (class, or 255 where the pixel does not count), or null: no loss, prediction only
void loss_pass(Ctx& c, const Geo& g, const ZSrc& zs, const uint8_t* labels8, const uint8_t* pixel_weights,
               const float* T, uint8_t* pred, float* slots, float* loss_part, unsigned long long* conf, bool grad,
               const CountSum* count = nullptr);

// k_update.hip
// (every per-head quantity below -- parameters, optimiser state, partial gradients, weight copies,
//  the caller's vectors -- holds Geo::heads() blocks; the kernels take the head from blockIdx.y)
// One Adam step's constants, prepared on the host in double precision:
//   theta <- theta - step_scale * m / (sqrt(v) * inv_sqrt_bc2 + eps),
//   step_scale = lr / (1 - beta1^t),  inv_sqrt_bc2 = 1 / sqrt(1 - beta2^t).
struct AdamStep { float beta1, beta2, one_minus_beta1, one_minus_beta2, eps, step_scale, inv_sqrt_bc2; };
void call_begin(Ctx& c, const Plan& p, char* ws, const void* features, int feat_dtype, const float* head_params,
                bool w1t, const int32_t* labels, const uint8_t* pixel_weights, const ZeroList& zero,
                const float* vel = nullptr, const float* vel2 = nullptr);
// blocks of the label role of that launch, in the order of the frames; each leaves its pixel count (weight sum)
int label_blocks(const Geo& g);
void step_end(Ctx& c, const Plan& p, char* ws, float lr, float mu, const AdamStep* adam, bool finish, float* loss_out,
              double* miou_out, long long* conf_out, bool w1t = false, float* save_old = nullptr);
// arguments of the bookkeeping role; miou_host / token_host / token as for finish_pass
FinishArgs finish_args(const Plan& p, char* ws, float* loss_out, double* miou_out, long long* conf_out,
                       double* miou_host = nullptr, unsigned long long* token_host = nullptr,
                       unsigned long long token = 0);
// miou_host: host memory the device can write (or null) that also receives the per-frame metric,
// each value followed by `token` in token_host (a release store at system scope)
void finish_pass(Ctx& c, const Plan& p, char* ws, float* loss_out, double* miou_out, long long* conf_out,
                 float* ext_out = nullptr, double* miou_host = nullptr, unsigned long long* token_host = nullptr,
                 unsigned long long token = 0, float* out_vel = nullptr, float* out_vel2 = nullptr);
void confusion_and_miou(Ctx& c, const uint8_t* pred, const int32_t* labels, long long P, int C, int ignore,
                        long long* conf, double* miou);

// k_weights.hip
void object_weights(Ctx& c, const int32_t* labels, int n, int H, int W, int C, int background, int ignore, int radius,
                    int factor, uint8_t* out);

}  // namespace st
