// Loss weights from the teacher's label map (Section 5.2: the cross-entropy of pixels near and
// within non-background objects is scaled by a factor; "near" = within `radius` pixels along x
// and along y).  One launch, one pass over the labels: 4 bytes read and 1 byte written per pixel.
//
// A block owns a tile of TH rows x 256 columns.  The object mask lives in LDS as a bit matrix,
// one 64-bit word per 64 consecutive pixels of a row: a wavefront loads 64 consecutive labels (one
// coalesced 256-byte read) and a single ballot turns them into a word.  The tile's mask is taken
// with `radius` more rows above and below and with the `radius` pixels on either side (one more
// load per row: the lanes that would hold them in the neighbouring words, right-hand ones first),
// then spread along x with shifts (bits cross word boundaries through the neighbouring words;
// radius <= 32 < 64, so one neighbour per side is enough), then along y by OR-ing 2 radius + 1
// rows.  Pixels outside the frame hold no object.  Each thread finally writes TH / 16 times four pixels.
//
// Bound by one trip to memory per block and by the instructions around its loads, so blocks are sized for one round over the chip: 32 rows
// where the frame makes at least 256 such tiles, else 16.  1920 x 1080,
// radius 4: 10.6 -> 6.8 us (16-row tiles, six words a row and a bounds test and a division per load before).
#include "st_common.hpp"
#include "st_kernels.hpp"

namespace st {

constexpr int OW_WORDS = 4;                  // 64-pixel words of a tile row
constexpr int OW_TW = 64 * OW_WORDS;         // columns of a tile
constexpr int OW_THREADS = 1024;
constexpr int OW_ROWS = 3;                   // rows a wavefront keeps in flight
static_assert(ST_OBJECT_WEIGHTS_MAX_RADIUS <= 32, "one neighbouring word per side; both sides in one load");

template <int TH>
__global__ void __launch_bounds__(OW_THREADS)
k_object_weights(const int32_t* __restrict__ labels, int H, int W, int C, int background, int ignore, int radius,
                 int factor, uint8_t* __restrict__ out)
{
    constexpr int ROWS = TH + 2 * ST_OBJECT_WEIGHTS_MAX_RADIUS;       // most mask rows a tile looks at
    __shared__ unsigned long long obj[ROWS * (OW_WORDS + 1)];         // object bits; word 4: the pixels beside the tile
    __shared__ unsigned long long hor[ROWS * OW_WORDS];               // spread along x
    __shared__ unsigned long long ver[TH * OW_WORDS];                 // and along y
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x0 = blockIdx.x * OW_TW, y0 = blockIdx.y * TH;
    const size_t frame = (size_t)blockIdx.z * H * W;
    const int rows = TH + 2 * radius;

    // object bits of rows y0 - radius .. y0 + TH + radius - 1: a wavefront takes every sixteenth row, OW_ROWS of
    // them in flight (with a radius of up to 8 that is all it has to load: one round trip to memory).
    // Loads are unconditional, from clamped addresses; what lies off the frame is masked out of the ballots,
    // which are scalars, and so is everything that depends on the row.
    constexpr int WAVES = OW_THREADS / 64, WORDS = OW_WORDS + 1;
    int xi[WORDS];
    unsigned long long on[WORDS];
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        // (the last word: lanes 0 .. radius - 1 hold the pixels right of the tile, lanes 64 - radius .. 63 those left of it)
        const int x = x0 + (w < OW_WORDS ? 64 * w + lane : lane < 32 ? OW_TW + lane : lane - 64);
        on[w] = __ballot(x >= 0 && x < W && (w < OW_WORDS || lane < radius || lane >= 64 - radius));
        xi[w] = min(max(x, 0), W - 1);
    }
    const int32_t* lab = labels + frame;
    for (int r0 = wave; r0 < rows; r0 += OW_ROWS * WAVES) {
        int v[OW_ROWS][WORDS];
#pragma unroll
        for (int k = 0; k < OW_ROWS; ++k) {
            const int y = min(max(y0 - radius + r0 + k * WAVES, 0), H - 1);
#pragma unroll
            for (int w = 0; w < WORDS; ++w) v[k][w] = (lab + (size_t)y * W)[xi[w]];
        }
#pragma unroll
        for (int k = 0; k < OW_ROWS; ++k) {
            const int row = r0 + k * WAVES, y = y0 - radius + row;
            const bool in = y >= 0 && y < H;
#pragma unroll
            for (int w = 0; w < WORDS; ++w) {
                const unsigned long long m = __ballot((unsigned)v[k][w] < (unsigned)C) & __ballot(v[k][w] != background) &
                                             __ballot(v[k][w] != ignore) & on[w];
                if (row < rows && lane == 0) obj[row * WORDS + w] = in ? m : 0ull;
            }
        }
    }
    __syncthreads();

    // bit x of the result = OR of bits x - radius .. x + radius
    for (int j = threadIdx.x; j < rows * OW_WORDS; j += OW_THREADS) {
        const int row = j / OW_WORDS, word = j - row * OW_WORDS;
        const unsigned long long* o = obj + row * (OW_WORDS + 1);
        // (the word beside the tile serves as the left neighbour of word 0 and the right one of word 3)
        const unsigned long long left = o[word > 0 ? word - 1 : OW_WORDS], mid = o[word], right = o[word + 1];
        unsigned long long h = mid;
        for (int s = 1; s <= radius; ++s)
            h |= (mid >> s) | (right << (64 - s)) | (mid << s) | (left >> (64 - s));
        hor[j] = h;
    }
    __syncthreads();

    if (threadIdx.x < TH * OW_WORDS) {
        const int row = threadIdx.x / OW_WORDS, word = threadIdx.x - row * OW_WORDS;
        unsigned long long v = 0;
        for (int d = 0; d <= 2 * radius; ++d) v |= hor[(row + d) * OW_WORDS + word];
        ver[threadIdx.x] = v;
    }
    __syncthreads();

    // four consecutive pixels per thread and trip: one 4-byte store where the address allows it
#pragma unroll
    for (int t = 0; t < TH / 16; ++t) {
        const int row = t * 16 + threadIdx.x / (OW_TW / 4), quad = threadIdx.x % (OW_TW / 4);
        const int y = y0 + row, x = x0 + 4 * quad;
        if (y < H && x < W) {
            const unsigned int bits = (unsigned int)(ver[row * OW_WORDS + (quad >> 4)] >> (4 * (quad & 15))) & 15u;
            uint8_t* dst = out + frame + (size_t)y * W + x;
            unsigned int packed = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) packed |= (unsigned int)(((bits >> i) & 1u) ? factor : 1) << (8 * i);
            if (x + 4 <= W && ((uintptr_t)dst & 3) == 0) {
                *(unsigned int*)dst = packed;
            } else {
                for (int i = 0; i < 4 && x + i < W; ++i) dst[i] = (uint8_t)(packed >> (8 * i));
            }
        }
    }
}

void object_weights(Ctx& c, const int32_t* labels, int n, int H, int W, int C, int background, int ignore, int radius,
                    int factor, uint8_t* out)
{
    const int cols = cdiv(W, OW_TW);
    if ((long long)cols * cdiv(H, 32) * n >= 256)
        ST_LAUNCH(c, "object_weights", k_object_weights<32>, dim3(cols, cdiv(H, 32), n), dim3(OW_THREADS), 0, labels, H, W, C, background,
                  ignore, radius, factor, out);
    else
        ST_LAUNCH(c, "object_weights", k_object_weights<16>, dim3(cols, cdiv(H, 16), n), dim3(OW_THREADS), 0, labels, H, W, C, background,
                  ignore, radius, factor, out);
}

}  // namespace st
