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
// vectors of the caller that overlap (their order counts); else this rides on the last launch of a call.  Thread x walks the
// caller's index (internal_index), so that the scattered side is the reads.
__global__ void __launch_bounds__(256)
k_permute_params(const float* __restrict__ src, float* __restrict__ dst, ParamOffsets po,
                 FastDiv by_in1, FastDiv by_in2, size_t head_stride)
{
    const unsigned x = blockIdx.x * 256 + threadIdx.x;
    // one head per blockIdx.y: internal blocks head_stride floats apart, external ones back to back
    if (x < po.total) dst[blockIdx.y * po.total + x] = src[blockIdx.y * head_stride + internal_index(po, by_in1, by_in2, x)];
}

void permute_params(Ctx& c, const Plan& p, const float* src, float* dst)
{
    ST_LAUNCH(c, "params_from_internal", k_permute_params, dim3(cdiv(p.po.total, 256), p.g.heads()), dim3(256), 0, src, dst,
              p.po, fast_div(p.g.c_in), fast_div(p.g.c1), p.head_stride);
}

}  // namespace st
