// The list of regions to clear, and the permutation from the internal parameter order ([o][kh][kw][i]) to the
// caller's (OIHW) in a launch of its own.
#include "st_kernels.hpp"
#include "st_mfma.hpp"

namespace st {

// (all workspace regions are 16-byte aligned and padded to 16 bytes)
void ZeroList::add(void* p, size_t bytes, int count, size_t stride_bytes)
{
    if (bytes == 0 || count == 0) return;
    if (n >= MAX) { overflow = true; return; }
    ptr[n] = (char*)p;
    stride[n] = stride_bytes;
    n16[n] = (unsigned)((bytes + 15) / 16);
    per[n] = (int)((n16[n] + ZERO_PER_BLOCK - 1) / ZERO_PER_BLOCK);
    first[n + 1] = first[n] + per[n] * count;
    ++n;
}

// One vector out of the workspace: for the calls with loop exits, where the host decides what is handed back, and for
// vectors of the caller that overlap (their order counts); else this rides on the last launch of a call.  Thread j walks the internal index; inside a 3x3 weight block
//   internal (o*9 + tap)*ci + i   <->   external (o*ci + i)*9 + tap.
__global__ void __launch_bounds__(256)
k_permute_params(const float* __restrict__ src, float* __restrict__ dst, ParamOffsets po,
                 int ci1, int ci2, size_t head_stride)
{
    const size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= po.total) return;
    // one head per blockIdx.y: internal blocks head_stride floats apart, external ones back to back
    src += blockIdx.y * head_stride;
    dst += blockIdx.y * po.total;
    size_t e = j;
    if (j < po.b1) {
        const size_t r = j - po.W1;
        const size_t i = r % ci1, tap = (r / ci1) % 9, o = r / ((size_t)ci1 * 9);
        e = po.W1 + (o * ci1 + i) * 9 + tap;
    } else if (j >= po.W2 && j < po.b2) {
        const size_t r = j - po.W2;
        const size_t i = r % ci2, tap = (r / ci2) % 9, o = r / ((size_t)ci2 * 9);
        e = po.W2 + (o * ci2 + i) * 9 + tap;
    }
    dst[e] = src[j];
}

void permute_params(Ctx& c, const Plan& p, const float* src, float* dst)
{
    ST_LAUNCH(c, "params_from_internal", k_permute_params, dim3(cdiv(p.po.total, 256), p.g.heads()), dim3(256), 0, src, dst,
              p.po, p.g.c_in, p.g.c1, p.head_stride);
}

}  // namespace st
