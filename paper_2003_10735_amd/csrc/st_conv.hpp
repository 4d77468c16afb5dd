// Arguments of the bfloat16 3x3 convolution kernels (k_conv_mfma.hip: small tiles, k_conv_wide.hip: large ones).
#pragma once
#include "st_mfma.hpp"

namespace st {

struct ConvArgs {
    const bf16* X;      // [PP][cin] position-major, guards before/after
    const bf16* Wq;     // fragment order, see wfrag_index(): rows = cout, K = cin
    const float* bias;  // EPI 0, 2
    const bf16* mask;   // EPI 1: activation whose sign gates the gradient, [PP][cout]
    bf16* Y;            // [PP][cout] or nullptr
    bf16* YT;           // channel-major copy, blocked layout of xt_index(), or nullptr
    // EPI 2: the 1x1 classifier rides along.  Every block adds its channels' share of the
    // logits of its positions: zpart[64 channels][padded position][zpitch classes] float32 (zpitch =
    // the class count rounded up to a multiple of four); the consumer adds the shares and
    // the bias.
    const bf16* W3q;    // [n_cls][cout] bfloat16
    float* zpart;
    int n_cls, zpitch;
    // EPI 3: the plain sums go, as float32, straight to a dense [n][cout][h][w] tensor
    float* dense; int dense_c;   // (channels of that tensor: cout without the padding)
    int PP, Hp, Wp, h, w, cin, cout, PPT, guard;
    int m_tiles, n_tiles, tiles_per_xcd;
    FastDiv by_n_tiles, by_grp_tiles, by_frame, by_row;     // (n_tiles; grp_tiles; Hp * Wp; Wp)
    // Several heads: positions [k * grp_pp, (k + 1) * grp_pp) use weight set k (Wq, bias and W3q
    // advance by wq_stride, bias_stride, w3_stride elements per set); position tiles are counted
    // per set (grp_tiles each) so that no tile mixes two sets.  One head: grp_pp = PP.
    int grp_pp, grp_tiles;
    size_t wq_stride, bias_stride, w3_stride;
};

// where padded position mp lies: the frame, and whether it is a cell of its grid (row y - 1, column x - 1)
struct ConvCell { int img, y, x; bool inside; };
__device__ __forceinline__ ConvCell conv_cell(const ConvArgs& a, int mp, int m_end)
{
    ConvCell c;
    c.img = fast_quot(mp, a.by_frame);
    const int rr = mp - c.img * (int)a.by_frame.d;
    c.y = fast_quot(rr, a.by_row); c.x = rr - c.y * (int)a.by_row.d;
    c.inside = mp < m_end && c.y >= 1 && c.y <= a.h && c.x >= 1 && c.x <= a.w;
    return c;
}

// Positions x channels of a block's tile: 64 channels name the kernel of k_conv_mfma.hip (32, 64 or 128 positions), 128 that of k_conv_wide.hip.
struct ConvTile { int bm, bn; };
ConvTile conv_tile(const Geo& g, int cin, int cout);
void conv3x3_wide(Ctx& c, const char* name, ConvArgs a, int epi, int heads);

}  // namespace st
