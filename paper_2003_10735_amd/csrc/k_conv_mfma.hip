// 3x3 convolution (forward, and data-gradient as a forward with mirrored taps) as an implicit
// GEMM on the gfx950 matrix cores: bfloat16 operands, float32 accumulation
// (v_mfma_f32_32x32x16_bf16).
//
//   out[mp][n] = epi( sum_{kh,kw,c} X[mp + (kh-1)*Wp + (kw-1)][c] * W[n][kh*3+kw][c] )
//
// X is position-major on the zero-padded grid, so a tap is a constant row offset and the GEMM's
// M index can simply walk the padded positions mp = 0 .. PP-1 linearly (results at border
// positions are forced to zero, which keeps the border of the output zero as well).  Guard rows
// in front of and behind every activation buffer make all reads in-bounds without tests.
//
// Block = 512 threads = 8 wavefronts, tile = 128 positions x 64 output channels.  A tile is
// small (every byte staged is used only a few times), and the matrix cores, the LDS read path,
// the vector-memory path and plain instruction issue are all close to full in the K loop; so the
// two operands take different routes and the loop is written to issue as little as possible:
//   * the weights are the MFMA A operand (rows = output channels) and never touch LDS: they are
//     kept in memory in fragment order (wfrag_index), so a wavefront fetches the fragment it
//     needs with one coalesced 1 KB buffer load straight into the operand registers (buffer
//     descriptor + fixed lane offset + one scalar offset per stage: no address arithmetic), and
//     no two wavefronts of a block need the same fragment;
//   * the activations are the B operand (columns = positions) and go through LDS, because the
//     three taps kw = 0,1,2 of a kernel row read the same slab at row offsets 0,1,2.  They are
//     loaded from memory directly into LDS (no registers, no LDS store instructions).
// Wavefront (wn, kgrp): output channels 32 wn .. +31 of the tile, all 128 positions (four
// accumulator tiles), and of every 64-channel stage the 16 input channels 16 kgrp .. +15.  The
// four partial sums per output are exchanged once, through LDS, after the K loop: wavefront
// (wn, kgrp) ends up owning positions 32 kgrp .. +31 and adds the partials in ascending kgrp.
// Grids that leave compute units without a block run tiles of 64 or 32 positions (MB = 2, 1; the rule is conv_tile's): the same
// wavefronts, channels and sums, two or one accumulator tiles each, and an owner of 8 or 4 of a tile's 16 registers.
// K loop: stages of (one kernel row kh) x (64 input channels): 130 activation rows in LDS (the
// tile's rows shifted by kh, plus one on each side) of 128 bytes, their 16-byte chunks swizzled
// by the row number so that the fragment reads of 16 consecutive rows spread over all banks.  Three
// slabs and three sets of weight registers rotate: loads run two stages ahead of the matrix cores.
// (Tiles of 32 positions: nine slabs, a barrier every three stages; activations run six stages ahead, weights two.)
//
// A lane owns 4 consecutive output channels of one position per register group, which packs
// into one 8-byte LDS write in the epilogue.  The epilogue stages the tile in LDS and writes it
// twice with 16-byte stores: position-major (input of the next convolution) and channel-major
// (operand of the weight-gradient kernel).  For the layer that feeds the 1x1 classifier the
// staged tile is also multiplied with the classifier's weights (16 more MFMAs per block), which
// saves the classifier a launch and a pass over the activations.
#include <type_traits>

#include "st_conv.hpp"
#include "st_kernels.hpp"

namespace st {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int CV_BN = 64;
constexpr int CV_BK = 64;
constexpr int CV_NBUF = 3;          // sets of activation slabs in LDS (ConvLds::PER slabs each): one in use, two on their way
constexpr int CV_OLD = CV_BN + 8;   // pitch of the staged output tile
// Tiles of 32 MB positions: 128, or 64 or 32 where those find a compute unit each of their own (conv_tile).
template <int MB>
struct ConvLds {
    static constexpr int BM = 32 * MB, ROWS = BM + 2, SLAB = ROWS * CV_BK * 2;       // one slab: BM + 2 rows of 64 channels, unpadded
    // dynamic LDS: the activation slabs, whose room the staged output tile takes afterwards, and behind them the exchanged partial
    // sums (8 owners x 3 sources x 4 MB registers x 64 lanes, float32), which are written while the last slab is still read
    static constexpr int PER = MB == 1 ? 3 : 1;           // stages between two barriers, whose slabs rotate together
    static constexpr size_t SLABS = (size_t)CV_NBUF * PER * SLAB, BYTES = SLABS + (size_t)8 * 3 * 4 * MB * 64 * sizeof(float);
    static_assert((size_t)BM * CV_OLD * sizeof(bf16) <= SLABS && BYTES <= 160 * 1024, "LDS buffers fit");
};

// TAG only gives every call site (layer 1 forward, layer 2 forward, layer 2 data-gradient) a
// kernel symbol of its own, so that profiles list them separately.
template <int EPI, int TAG, int MB>
__global__ void __launch_bounds__(512) k_conv3x3_mfma(ConvArgs a)
{
    constexpr int NT = 512;                // threads per block
    constexpr int BM = ConvLds<MB>::BM, XS_BYTES = ConvLds<MB>::SLAB;
    constexpr int NR = 4 * MB;             // registers (of 16 per 32 x 32 sums) of an owner: a wavefront's MB tiles are four parts
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    // smem_raw during the K loop: [CV_NBUF * PER][BM + 2][128 bytes], chunks swizzled

    // (what the first loads need, in one trip for the arguments: left to itself the compiler asks for some of it only
    //  behind the question whether the block has a tile)
    asm volatile("" ::"s"(a.tiles_per_xcd), "s"(a.m_tiles), "s"(a.n_tiles), "s"(a.by_n_tiles.m), "s"(a.by_grp_tiles.m), "s"(a.grp_tiles), "s"(a.grp_pp),
                 "s"(a.X), "s"(a.Wq), "s"(a.wq_stride), "s"(a.cin), "s"(a.Wp));
    // XCD-aware tile order: consecutive blocks go to different XCDs, so give each XCD a
    // contiguous run of position tiles (neighbours share activation rows in that XCD's L2)
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int tile = xcd * a.tiles_per_xcd + slot;
    if (slot >= a.tiles_per_xcd || tile >= a.m_tiles * a.n_tiles) return;
    const int mt = fast_quot(tile, a.by_n_tiles), nt = tile - mt * a.n_tiles;
    const int grp = fast_quot(mt, a.by_grp_tiles);
    const int m0 = grp * a.grp_pp + (mt - grp * a.grp_tiles) * BM, n0 = nt * CV_BN;
    const int m_end = (grp + 1) * a.grp_pp;     // results from here on belong to another tile

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kgrp = wave >> 1;
    const int l32 = lane & 31, lhi = lane >> 5;

    // The sums in four parts: part s goes to the wavefront of K group kgrp ^ s, and part 0 is the one this wavefront owns in the
    // end.  MB = 4: part s is acc[s], 32 channels of positions 32 (s ^ kgrp) .. + 31.  With fewer positions a part is a half or a quarter of
    // a tile's channels: acc[j] are positions 32 (j ^ kgrp % MB) .. + 31, and row m of the MFMAs is channel m ^ row_x.
    const int row_x = MB == 4 ? 0 : MB == 2 ? (kgrp >> 1) * 16 : kgrp * 8;
    f32x16 acc[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

    const int c_chunks = a.cin / CV_BK;
    const int n_stages = 3 * c_chunks;
    const int kfr = a.cin >> 4;                                   // 16-channel fragments per tap
    const int nb = (n0 >> 5) + wn;                                // this wavefront's block of 32 output channels

    u32x4 wr[3][3];          // weight fragments of the three taps of a stage: in use, and two stages ahead

    // ---- activations: global memory -> LDS without passing through registers.  A wavefront-wide
    // 16-byte load puts lane l's bytes at (LDS base in M0) + 16 l, so one instruction fills eight
    // consecutive 128-byte rows (64 channels) of a slab.  Rows filled this way cannot be padded;
    // instead the 16-byte chunk c of row r is kept at chunk position c ^ ((r >> 1) & 7).  LDS
    // serves 16 lanes of a 16-byte read per cycle (64 banks): the 16 consecutive rows they read
    // are 8 even rows (banks 0-31) and 8 odd rows (banks 32-63), and within each group the eight
    // values of (r >> 1) & 7 differ, so the reads spread over all banks just as padded rows
    // would.  The lane that fills position pc of row r fetches chunk pc ^ ((r >> 1) & 7).
    // Wavefront w fills rows 8w .. 8w+7 and, of 130, 64+8w .. 64+8w+7; wavefront 0 also rows 128, 129.  The short stages of small
    // tiles cannot afford that wavefront 0 so has one load more to wait for than the others: there every wavefront that fills rows (of
    // 34 the first four) also fills the two behind BM, all with the same bytes.  (With 130 rows the eight loads cost more: key frame at 90 x 160
    // cells 641 -> 649 us.)
    // The loads are written in assembly: the compiler would order every barrier behind all
    // outstanding loads of this kind, while the pipeline below needs two stages or more in flight.
    // (M0 is a reserved register for this compiler: it never allocates a value to it, sets it
    //  right before each instruction of its own that reads it, and rejects it in an asm clobber
    //  list ("inline asm clobber list contains reserved registers: m0") -- so the statement
    //  below cannot declare the write and does not need to: nothing of the compiler's lives in M0
    //  across it, and each statement sets M0 itself before the one load that reads it.  One wait
    //  state separates the scalar write of M0 from that load.)
    const int lrow = lane >> 3, lpc = lane & 7;
    const int sw01 = (4 * wave + (lrow >> 1)) & 7, sw2 = lrow >> 1;          // (row >> 1) & 7 of the rows filled
    const int xo0 = ((wave * 8 + lrow) * a.cin + ((lpc ^ sw01) << 3)) * 2;   // byte offsets inside a slab
    const int xo1 = xo0 + 64 * a.cin * 2;
    const int xo2 = ((BM + lrow) * a.cin + ((lpc ^ sw2) << 3)) * 2;
    const bf16* xg = a.X + ((long long)m0 - 1 - a.Wp) * a.cin;               // first row of the kh = 0 slabs
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const unsigned wave_lds = __builtin_amdgcn_readfirstlane(wave * 1024);   // a scalar: it goes to M0
    // fragment reads: row 32 (J ^ kgrp % MB) + l32 + KW, chunk kgrp*2 + lhi
    int rd[3][MB];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw)
#pragma unroll
        for (int J = 0; J < MB; ++J)
            rd[kw][J] = (l32 + kw) * 128 + (((kgrp * 2 + lhi) ^ (((l32 + kw) >> 1) & 7)) << 4) + (J ^ (kgrp & (MB - 1))) * 4096;

    // The stage being fetched runs two ahead of the one being multiplied (activations of tiles of 32 positions: six).  Its operands are
    // addressed as (scalar base, advanced once per stage) + (per-lane byte offset, fixed), which
    // costs no vector instruction and two scalar ones per stage.
    const char* xsp = (const char*)xg;                                      // activations of the stage
    // (weights through a buffer descriptor: base in scalar registers, a fixed per-lane offset and
    //  a scalar offset per stage, so that a weight load needs no address arithmetic at all)
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.Wq + grp * a.wq_stride), 0, (int)(a.wq_stride * 2), 0x00020000);
    int w_soff = 0;                                                          // weights of the stage
    unsigned wv[3];
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) wv[kw] = (unsigned)((((nb * 9 + kw) * kfr + kgrp) * 512 + (lane ^ row_x) * 8) * 2);
    const long long x_step = CV_BK * 2, x_row = ((long long)a.Wp * a.cin - (c_chunks - 1) * CV_BK) * 2;
    const int w_step = (CV_BK / 16) * 512 * 2, w_row = (2 * kfr + CV_BK / 16) * 512 * 2;
    int f_cc = 0, x_cc = 0;
#define CV_FETCH_NEXT                                                                             \
    if (++f_cc == c_chunks) { f_cc = 0; xsp += x_row; w_soff += w_row; } else { xsp += x_step; w_soff += w_step; }
    // (small tiles, whose activations run further ahead than their weights)
#define CV_W_NEXT if (++f_cc == c_chunks) { f_cc = 0; w_soff += w_row; } else w_soff += w_step;
#define CV_X_NEXT if (++x_cc == c_chunks) { x_cc = 0; xsp += x_row; } else xsp += x_step;
#define CV_DMA(VOFF, LDSADDR)                                                                     \
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(VOFF), "s"(xsp), \
                 "s"(LDSADDR) : "memory");
    // (the same for lanes 0 .. 15 alone: every lane of the kernel is active here, before and behind)
#define CV_DMA2(VOFF, LDSADDR)                                                                    \
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, 0xffff\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1" ::"v"(VOFF), \
                 "s"(xsp), "s"(LDSADDR) : "memory");
#define CV_LOAD_X1(BUF, I)                                                                        \
    {                                                                                             \
        if ((I) == 0 && (MB > 1 || wave < 4)) CV_DMA(xo0, lds0 + (BUF) * XS_BYTES + wave_lds)     \
        if ((I) == 1 && MB == 4) CV_DMA(xo1, lds0 + (BUF) * XS_BYTES + 8192 + wave_lds)           \
        if ((I) == 2 && MB == 4 && wave == 0 && lane < 16) CV_DMA(xo2, lds0 + (BUF) * XS_BYTES + BM * 128) \
        if ((I) == 2 && (MB == 2 || (MB == 1 && wave < 4))) CV_DMA2(xo2, lds0 + (BUF) * XS_BYTES + BM * 128) \
    }
#define CV_LOAD_W(SET, KW) wr[SET][KW] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wv[KW], w_soff, 0);
#define CV_READ1(DST, J, BUF, KW)                                                                 \
    DST[J] = *(const bf16x8*)(smem_raw + (BUF) * XS_BYTES + rd[KW][J]);
#define CV_MMA1(SRC, J, SET, KW)                                                                  \
    acc[J] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wr[SET][KW]), SRC[J], acc[J], 0, 0, 0);
    // s_waitcnt vmcnt(N) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, no wait on the others)
#define CV_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | 0x0F70);
    // One stage out of LDS slab and weight register set B.  With FETCH, the activations and
    // weights of the stage two ahead start their way into slab / set (B + 2) % 3, which the stage
    // before this one used last; the loads are spread over the stage, one after every other
    // MFMA.  Before the barrier that ends the stage every wavefront waits until its own share of
    // the next stage's slab has landed: everything but the loads issued during this stage (three and CV_XL for the
    // slab; wavefront 0 of 130 rows has one more), or simply everything when the stage issued none.
    constexpr int CV_XL = 2;
#define CV_F __builtin_amdgcn_sched_barrier(0);
#define CV_STAGE(B, FETCH)                                                                        \
    if constexpr (MB == 4) {                                                                      \
        constexpr int N_ = ((B) + 2) % 3;                                                         \
        CV_READ1(xa, 0, B, 0) CV_READ1(xa, 1, B, 0) CV_READ1(xa, 2, B, 0) CV_READ1(xa, 3, B, 0)   \
        CV_READ1(xb, 0, B, 1) CV_F                                                                \
        CV_MMA1(xa, 0, B, 0) CV_F if (FETCH) CV_LOAD_W(N_, 0) CV_READ1(xb, 1, B, 1) CV_F          \
        CV_MMA1(xa, 1, B, 0) CV_F if (FETCH) CV_LOAD_W(N_, 1) CV_READ1(xb, 2, B, 1) CV_F          \
        CV_MMA1(xa, 2, B, 0) CV_F if (FETCH) CV_LOAD_W(N_, 2) CV_READ1(xb, 3, B, 1) CV_F          \
        CV_MMA1(xa, 3, B, 0) CV_F                                                                 \
        CV_MMA1(xb, 0, B, 1) CV_F if (FETCH) CV_LOAD_X1(N_, 0) CV_READ1(xa, 0, B, 2) CV_F         \
        CV_MMA1(xb, 1, B, 1) CV_F CV_READ1(xa, 1, B, 2) CV_F                                      \
        CV_MMA1(xb, 2, B, 1) CV_F if (FETCH) CV_LOAD_X1(N_, 1) CV_READ1(xa, 2, B, 2) CV_F         \
        CV_MMA1(xb, 3, B, 1) CV_F CV_READ1(xa, 3, B, 2) CV_F                                      \
        CV_MMA1(xa, 0, B, 2) CV_F if (FETCH) CV_LOAD_X1(N_, 2) CV_F                               \
        CV_MMA1(xa, 1, B, 2) CV_F                                                                 \
        CV_MMA1(xa, 2, B, 2) CV_F                                                                 \
        CV_MMA1(xa, 3, B, 2) CV_F                                                                 \
        if (FETCH) { CV_FETCH_NEXT CV_VMCNT(3 + CV_XL) } else { CV_VMCNT(0) }                     \
        __syncthreads();                                                                          \
    } else if constexpr (MB == 2) {                                                               \
        constexpr int N_ = ((B) + 2) % 3;                                                         \
        CV_READ1(xa, 0, B, 0) CV_READ1(xa, 1, B, 0) CV_READ1(xb, 0, B, 1)                         \
        CV_READ1(xb, 1, B, 1) CV_READ1(xc, 0, B, 2) CV_READ1(xc, 1, B, 2) CV_F                    \
        CV_MMA1(xa, 0, B, 0) CV_F if (FETCH) CV_LOAD_W(N_, 0) CV_F                                \
        CV_MMA1(xa, 1, B, 0) CV_F if (FETCH) CV_LOAD_W(N_, 1) CV_F                                \
        CV_MMA1(xb, 0, B, 1) CV_F if (FETCH) CV_LOAD_W(N_, 2) CV_F                                \
        CV_MMA1(xb, 1, B, 1) CV_F if (FETCH) CV_LOAD_X1(N_, 0) CV_F                               \
        CV_MMA1(xc, 0, B, 2) CV_F if (FETCH) CV_LOAD_X1(N_, 2) CV_F                               \
        CV_MMA1(xc, 1, B, 2) CV_F                                                                 \
        if (FETCH) { CV_FETCH_NEXT CV_VMCNT(3 + CV_XL) } else { CV_VMCNT(0) }                     \
        __syncthreads();                                                                          \
    }

    // The smallest tiles, three MFMAs a stage: three stages between two barriers, out of slabs cur, cur + 1, cur + 2; meanwhile the activations of
    // the stage six ahead start their way into slab far + B, which every wavefront has left behind the barrier.  A barrier and the first
    // reads behind it take longer than such a stage's MFMAs.  Calls, a barrier a stage -> this: 16 x 24 cells, 64 channels, 4 steps
    // 150.5 -> 148.5 us; 30 x 53, 256 -> 128 -> 128 209.2 -> 207.9, forward 22.7 -> 22.5; 60 x 107, 96 -> 48 -> 48 206.1 -> 204.4.  (Tiles of 64
    // positions lost 1 % that way: 60 x 107 cells, 256 -> 128 -> 128, forward 23.2 -> 23.5.  Their first barrier waits for three slabs.)
#define CV_SMALL(B, FETCH_W, FETCH_X)                                                             \
    {                                                                                             \
        constexpr int N_ = ((B) + 2) % 3;                                                         \
        CV_READ1(xa, 0, cur + B, 0) CV_READ1(xb, 0, cur + B, 1) CV_READ1(xc, 0, cur + B, 2) CV_F  \
        CV_MMA1(xa, 0, B, 0) CV_F                                                                 \
        if (FETCH_W) { CV_LOAD_W(N_, 0) CV_LOAD_W(N_, 1) } CV_F                                   \
        CV_MMA1(xb, 0, B, 1) CV_F                                                                 \
        if (FETCH_W) CV_LOAD_W(N_, 2) if (FETCH_X) CV_LOAD_X1(far + B, 0) CV_F                    \
        CV_MMA1(xc, 0, B, 2) CV_F                                                                 \
        if (FETCH_X) CV_LOAD_X1(far + B, 2) CV_F                                                  \
        if (FETCH_W) { CV_W_NEXT }                                                                \
        if (FETCH_X) { CV_X_NEXT }                                                                \
    }

    bf16x8 xa[MB], xb[MB], xc[MB];
    int cur = 0;             // first slab in use (other tiles: stays, their slabs rotate by number)
    if constexpr (MB > 1) {
        {
            // (activations first: the barrier waits for those of the first stage alone, everything but the loads behind them)
            CV_LOAD_X1(0, 0) CV_LOAD_X1(0, 1) CV_LOAD_X1(0, 2)
            CV_LOAD_W(0, 0) CV_LOAD_W(0, 1) CV_LOAD_W(0, 2)
            CV_FETCH_NEXT
            CV_LOAD_X1(1, 0) CV_LOAD_X1(1, 1) CV_LOAD_X1(1, 2)
            CV_LOAD_W(1, 0) CV_LOAD_W(1, 1) CV_LOAD_W(1, 2)
            CV_FETCH_NEXT
            CV_F
            CV_VMCNT(6 + CV_XL)
            __syncthreads();
        }
        // the number of stages is a multiple of three (three kernel rows): three stages per trip make
        // the LDS slab and the weight register set of every stage compile-time choices.  The last
        // three stages are written out: only the first of them still has something to fetch.
        for (int s = 0; s + 3 < n_stages; s += 3) {
            CV_STAGE(0, true)
            CV_STAGE(1, true)
            CV_STAGE(2, true)
        }
        CV_STAGE(0, true)
        CV_STAGE(1, false)
    } else {
        const int trips = c_chunks;       // (three stages each)
        int far = 6;
        {
            CV_LOAD_X1(0, 0) CV_LOAD_X1(0, 2) CV_X_NEXT
            CV_LOAD_X1(1, 0) CV_LOAD_X1(1, 2) CV_X_NEXT
            CV_LOAD_X1(2, 0) CV_LOAD_X1(2, 2) CV_X_NEXT
            CV_LOAD_W(0, 0) CV_LOAD_W(0, 1) CV_LOAD_W(0, 2) CV_W_NEXT
            CV_LOAD_W(1, 0) CV_LOAD_W(1, 1) CV_LOAD_W(1, 2) CV_W_NEXT
            CV_F
            if (trips > 1) {
                CV_LOAD_X1(3, 0) CV_LOAD_X1(3, 2) CV_X_NEXT
                CV_LOAD_X1(4, 0) CV_LOAD_X1(4, 2) CV_X_NEXT
                CV_LOAD_X1(5, 0) CV_LOAD_X1(5, 2) CV_X_NEXT
                CV_VMCNT(6 + 3 * CV_XL)
            } else { CV_VMCNT(6) }
            __syncthreads();
        }
        for (int t = 0; t + 2 < trips; ++t) {
            CV_SMALL(0, true, true)
            CV_SMALL(1, true, true)
            CV_SMALL(2, true, true)
            // (what follows the next three stages' activations: nine weight fragments and three stages' activations)
            CV_VMCNT(9 + 3 * CV_XL)
            __syncthreads();
            far = cur;
            cur = cur == 6 ? 0 : cur + 3;
        }
        if (trips > 1) {
            CV_SMALL(0, true, false)
            CV_SMALL(1, true, false)
            CV_SMALL(2, true, false)
            CV_VMCNT(9)
            __syncthreads();
            cur = cur == 6 ? 0 : cur + 3;
        }
        CV_SMALL(0, true, false)
        CV_SMALL(1, false, false)
    }
    // The last stage takes one accumulator tile behind the other, the tiles of other owners first, so that a finished tile is on its way
    // to LDS while the next one's MFMAs run.  (With the order of the first loads and the transposing reads below, launches before -> now: 90 x 160
    // cells, 256 -> 128 -> 128 13.2 -> 12.6, 9.6 -> 9.0, 9.6 -> 8.6 us; 60 x 107 11.6 -> 10.8, 8.05 -> 7.1.)
    // (red: [owner's K group][wn][part - 1][NR / 4 register groups][64 lanes][4])
    float* red = (float*)(smem_raw + ConvLds<MB>::SLABS) + wn * 3 * NR * 64 + lane * 4;
    // register groups Q0 .. Q1 - 1 of part S: those from Q of acc[J] on
#define CV_HAND(S, Q0, Q1)                                                                        \
    {                                                                                             \
        constexpr int J_ = (S) % MB, Q_ = (S) / MB * MB;                                          \
        float* dst_ = red + ((S) ^ kgrp) * 6 * NR * 64 + ((S) - 1) * NR * 64;                     \
        _Pragma("unroll") for (int q = Q0; q < Q1; ++q)                                           \
            *(f32x4*)(dst_ + q * 256) = f32x4{acc[J_][(Q_ + q) * 4], acc[J_][(Q_ + q) * 4 + 1], acc[J_][(Q_ + q) * 4 + 2], acc[J_][(Q_ + q) * 4 + 3]}; \
    }
    if constexpr (MB == 4) {
        CV_READ1(xa, 1, 2, 0) CV_READ1(xb, 1, 2, 1) CV_READ1(xc, 1, 2, 2) CV_READ1(xa, 2, 2, 0) CV_READ1(xb, 2, 2, 1) CV_READ1(xc, 2, 2, 2) CV_F
        CV_MMA1(xa, 1, 2, 0) CV_F CV_READ1(xa, 3, 2, 0) CV_F
        CV_MMA1(xb, 1, 2, 1) CV_F CV_READ1(xb, 3, 2, 1) CV_F
        CV_MMA1(xc, 1, 2, 2) CV_F CV_READ1(xc, 3, 2, 2) CV_F
        CV_MMA1(xa, 2, 2, 0) CV_F CV_READ1(xa, 0, 2, 0) CV_F
        CV_MMA1(xb, 2, 2, 1) CV_F CV_READ1(xb, 0, 2, 1) CV_F
        CV_MMA1(xc, 2, 2, 2) CV_F CV_READ1(xc, 0, 2, 2) CV_F
        CV_MMA1(xa, 3, 2, 0) CV_F
        CV_HAND(1, 0, 2) CV_F
        CV_MMA1(xb, 3, 2, 1) CV_F
        CV_HAND(1, 2, 4) CV_F
        CV_MMA1(xc, 3, 2, 2) CV_F
        CV_HAND(2, 0, 2) CV_F
        CV_MMA1(xa, 0, 2, 0) CV_F
        CV_HAND(2, 2, 4) CV_F
        CV_MMA1(xb, 0, 2, 1) CV_F
        CV_MMA1(xc, 0, 2, 2) CV_F
        CV_HAND(3, 0, 4)
    } else if constexpr (MB == 2) {
        // (parts 1 and 3 are halves of acc[1], part 2 the other half of acc[0])
        CV_READ1(xa, 1, 2, 0) CV_READ1(xb, 1, 2, 1) CV_READ1(xc, 1, 2, 2) CV_READ1(xa, 0, 2, 0) CV_READ1(xb, 0, 2, 1) CV_READ1(xc, 0, 2, 2) CV_F
        CV_MMA1(xa, 1, 2, 0) CV_F
        CV_MMA1(xb, 1, 2, 1) CV_F
        CV_MMA1(xc, 1, 2, 2) CV_F
        CV_MMA1(xa, 0, 2, 0) CV_F
        CV_HAND(1, 0, 2) CV_F
        CV_MMA1(xb, 0, 2, 1) CV_F
        CV_HAND(3, 0, 2) CV_F
        CV_MMA1(xc, 0, 2, 2) CV_F
        CV_HAND(2, 0, 2)
    } else {
        CV_READ1(xa, 0, cur + 2, 0) CV_READ1(xb, 0, cur + 2, 1) CV_READ1(xc, 0, cur + 2, 2) CV_F
        CV_MMA1(xa, 0, 2, 0)
        CV_MMA1(xb, 0, 2, 1)
        CV_MMA1(xc, 0, 2, 2)
        CV_HAND(1, 0, 1)
        CV_HAND(2, 0, 1)
        CV_HAND(3, 0, 1)
    }
#undef CV_HAND
#undef CV_STAGE
#undef CV_SMALL
#undef CV_FETCH_NEXT
#undef CV_W_NEXT
#undef CV_X_NEXT
#undef CV_LOAD_X1
#undef CV_LOAD_W
#undef CV_DMA
#undef CV_DMA2
#undef CV_READ1
#undef CV_MMA1
#undef CV_VMCNT
#undef CV_F

    // ---- what the epilogue needs from memory, on its way while the partial sums are exchanged (asked for behind the
    //      exchange, it cost every launch a memory latency of its own; with the divisions of block and cell indexes as
    //      products, 8-step key frame at 90 x 160 cells 656 -> 638 us, forward at 60 x 107 27.4 -> 26.4)
    const int p = (kgrp & (MB - 1)) * 32 + l32, mp = m0 + p;         // this lane's position behind the exchange
    const ConvCell cell = conv_cell(a, mp, m_end);
    const bool inside = cell.inside;
    const int c_own = wn * 32 + row_x + lhi * 4;                     // and its channels: + 8 rg .. + 3, rg < MB
    f32x4 bias[EPI == 0 || EPI == 2 ? MB : 1];
    bf16x4 mk[EPI == 1 ? MB : 1];
    u32x4 w3f[EPI == 2 ? 4 : 1];
#pragma unroll
    for (int rg = 0; rg < MB; ++rg) {
        const int c = n0 + c_own + rg * 8;
        if (EPI == 0 || EPI == 2) bias[rg] = *(const f32x4*)(a.bias + grp * a.bias_stride + c);
        if (EPI == 1) mk[rg] = *(const bf16x4*)(a.mask + (size_t)min(mp, m_end - 1) * a.cout + c);
    }
    // (classifier fragments: A operand, rows = classes, k = 16 channels of this tile)
    if (EPI == 2)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            w3f[ks] = *(const u32x4*)(a.W3q + grp * a.w3_stride + (size_t)min(l32, a.n_cls - 1) * a.cout + n0 + lhi * 8 + ks * 16);

    // ---- exchange of the partial sums: each part has gone to its owner, which adds the four in ascending source order
    __syncthreads();
    float mine[NR];
    {
        // the parts of the three other K groups, in ascending order
        const float* from = red + kgrp * 6 * NR * 64;
        f32x4 part[3][MB];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int k = i + (i >= kgrp ? 1 : 0);
#pragma unroll
            for (int q = 0; q < MB; ++q) part[i][q] = *(const f32x4*)(from + ((k ^ kgrp) - 1) * NR * 64 + q * 256);
        }
#define CV_PART(I) part[I][r >> 2][r & 3]
        if (kgrp < 2) {         // (first or second: the same sum)
#pragma unroll
            for (int r = 0; r < NR; ++r) mine[r] = ((CV_PART(0) + acc[0][r]) + CV_PART(1)) + CV_PART(2);
        } else if (kgrp == 2) {
#pragma unroll
            for (int r = 0; r < NR; ++r) mine[r] = ((CV_PART(0) + CV_PART(1)) + acc[0][r]) + CV_PART(2);
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) mine[r] = ((CV_PART(0) + CV_PART(1)) + CV_PART(2)) + acc[0][r];
        }
#undef CV_PART
    }

    if (EPI == 3) {
        // a lane holds NR channels of one position; for a fixed channel the 32 lanes of a half
        // wavefront are 32 consecutive positions, i.e. (inside one grid row) consecutive floats
        if (inside) {
            float* dst = a.dense + ((size_t)cell.img * a.dense_c * a.h + (cell.y - 1)) * a.w + (cell.x - 1);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int ch = n0 + c_own + (r >> 2) * 8 + (r & 3);
                if (ch < a.dense_c) dst[(size_t)ch * a.h * a.w] = mine[r];
            }
        }
        return;
    }

    // ---- epilogue: bias + ReLU (forward) or ReLU mask (data-gradient), zero outside the grid,
    //      round to bfloat16, stage the tile in LDS as [position][channel]
    bf16* Os = (bf16*)smem_raw;     // [BM][CV_OLD], where the slabs were
#pragma unroll
    for (int rg = 0; rg < MB; ++rg) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = mine[rg * 4 + e];
            if (EPI == 1) v = (float)mk[rg][e] > 0.f ? v : 0.f;
            else v = fmaxf(v + bias[rg][e], 0.f);
            o[e] = (bf16)(inside ? v : 0.f);
        }
        *(bf16x4*)(Os + p * CV_OLD + c_own + rg * 8) = o;
    }
    __syncthreads();
    if (EPI == 2 && wave < MB) {
        // D[class][position] for positions 32 wave .. +31 over the tile's 64 channels
        f32x16 zacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) zacc[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bf16x8 xf = *(const bf16x8*)(Os + (wave * 32 + l32) * CV_OLD + ks * 16 + lhi * 8);
            const u32x4 wf = l32 < a.n_cls ? w3f[ks] : u32x4{0u, 0u, 0u, 0u};
            zacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf), xf, zacc, 0, 0, 0);
        }
        const int zp = m0 + wave * 32 + l32;
        if (zp < m_end) {
            // (a lane holds classes 8 gq + 4 lhi .. + 3; the groups beyond the classes are padding)
            float* zrow = a.zpart + ((size_t)nt * a.PP + zp) * a.zpitch + lhi * 4;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq)
                if (gq * 8 + lhi * 4 < a.zpitch)
                    *(f32x4*)(zrow + gq * 8) = f32x4{zacc[gq * 4], zacc[gq * 4 + 1], zacc[gq * 4 + 2], zacc[gq * 4 + 3]};
        }
    }
    if (a.Y) {
        // position-major: 16 bytes = 8 channels of one position
#pragma unroll
        for (int q = tid; q < BM * (CV_BN / 8); q += NT) {
            const int p = q / (CV_BN / 8), part = q % (CV_BN / 8);
            if (m0 + p < m_end)
                store_through(a.Y + (size_t)m0 * a.cout + n0, (unsigned)(p * a.cout + part * 8) * 2, *(const u32x4*)(Os + p * CV_OLD + part * 8));
        }
    }
    if (a.YT) {
        // channel-major: 16 bytes = 8 consecutive positions of one channel, a wavefront two such groups of 32
        // channels, through the transposing LDS read: in a group of 16 lanes, lane r names (position r / 4,
        // channels 4 (r % 4) .. + 3) and lane i receives channel i of four consecutive positions
#pragma unroll
        for (int u = wave; u < 4 * MB; u += 8) {
            const int pg = (u >> 1) * 2 + lhi, c = (u & 1) * 32;
            const bf16* row = Os + (pg * 8 + ((lane & 15) >> 2)) * CV_OLD + c + (lane & 16) + 4 * (lane & 3);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)row);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(row + 4 * CV_OLD));
            const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            if (m0 + pg * 8 < m_end)
                store_through(a.YT + xt_index(n0 + c, a.guard + m0 + (u >> 1) * 16, a.PPT / 8), lhi * 512 + l32 * 16, __builtin_bit_cast(u32x4, v));
        }
    }
}

// (cin and cout are multiples of 64 here: Geo::ki, k1, k2)
// epi 0: Y = relu(conv + bias) (layer 1); epi 2: the same, and with W3q / zpart the block also leaves its share
// of the classifier's logits (layer 2); epi 1: Y = conv * [mask > 0]; epi 3: the plain
// sums as float32 to the dense tensor `dense` [n][cout][h][w]
void conv3x3_mfma(Ctx& c, const char* name, const Plan& p, const bf16* X, const bf16* Wq, const float* bias,
                  const bf16* mask, bf16* Y, bf16* YT, int cin, int cout, int epi, const bf16* W3q,
                  float* zpart, float* dense)
{
    const Geo& g = p.g;
    ConvArgs a;
    a.X = X; a.Wq = Wq; a.bias = bias; a.mask = mask; a.Y = Y; a.YT = YT;
    a.W3q = W3q; a.zpart = zpart; a.n_cls = p.g.C; a.zpitch = (p.g.C + 3) / 4 * 4; a.dense = dense; a.dense_c = g.c_in;
    a.PP = p.g.padded_positions(); a.Hp = p.g.Hp; a.Wp = p.g.Wp; a.h = p.g.h; a.w = p.g.w;
    a.cin = cin; a.cout = cout;
    a.PPT = p.PPT; a.guard = p.guard;
    a.by_frame = g.by_frame; a.by_row = g.by_row;
    // several heads: one weight set per frame (Wq holds them back to back, the biases sit
    // head_stride floats apart inside the parameter vectors, W3q back to back)
    a.grp_pp = g.grouped ? g.Hp * g.Wp : a.PP;
    a.wq_stride = (size_t)cin * cout * 9;
    a.bias_stride = p.head_stride;
    a.w3_stride = (size_t)g.C * cout;
    const ConvTile t = conv_tile(g, cin, cout);
    if (t.bn != CV_BN) { conv3x3_wide(c, name, a, epi, g.heads()); return; }
    a.grp_tiles = cdiv(a.grp_pp, t.bm);
    a.m_tiles = g.heads() * a.grp_tiles;
    a.n_tiles = cout / CV_BN;
    a.by_n_tiles = fast_div(a.n_tiles); a.by_grp_tiles = fast_div(a.grp_tiles);
    const int tiles = a.m_tiles * a.n_tiles;
    a.tiles_per_xcd = cdiv(tiles, 8);
    const dim3 grid(a.tiles_per_xcd * 8);
    // tag 1: layer-1 forward, 2: layer-2 forward, 3: layer-2 data-gradient, 4: layer-1 data-gradient
    auto go = [&](auto kernel, size_t smem) {
        ensure_dynamic_lds((const void*)kernel, smem);
        ST_LAUNCH(c, name, kernel, grid, dim3(512), smem, a);
    };
    auto tiles_of = [&](auto mb) {
        constexpr int MB = decltype(mb)::value;
        if (epi == 3) go(k_conv3x3_mfma<3, 4, MB>, ConvLds<MB>::BYTES);
        else if (epi == 1) go(k_conv3x3_mfma<1, 3, MB>, ConvLds<MB>::BYTES);
        else if (epi == 2) go(k_conv3x3_mfma<2, 2, MB>, ConvLds<MB>::BYTES);
        else go(k_conv3x3_mfma<0, 1, MB>, ConvLds<MB>::BYTES);
    };
    if (t.bm == 128) tiles_of(std::integral_constant<int, 4>{});
    else if (t.bm == 64) tiles_of(std::integral_constant<int, 2>{});
    else tiles_of(std::integral_constant<int, 1>{});
}

}  // namespace st
