// Bookkeeping of a forward pass (role (3) of the step-closing kernel): per-frame mean IoU from the
// confusion counts, the tile losses added in a fixed order.  A header of its own because the role
// also rides on other launches (the classifier's backward kernel in the early-exit form).
#pragma once
#include "st_common.hpp"

namespace st {

struct FinishArgs {
    const float* loss_part; int n_part; const unsigned long long* n_valid; unsigned long long* conf;
    int n, C; float* loss_out; double* miou_a; double* miou_b; long long* conf_out;
    // per head (blockIdx.y): fph frames and pph tile losses; one head owns all of them
    int fph, pph;
    // early-exit form only: host memory that also receives the per-frame metric, each value followed by
    // the pass's token in token_c (or null)
    double* miou_c; unsigned long long* token_c; unsigned long long token;
};

// (EE: the early-exit form's extra -- the host copy of the metric -- is compiled in; NT: threads of the
// block, 256 of which add the tile losses whatever NT is, so that the order of the sum is one)
//
// Either kind of block is one chain of dependent steps on an otherwise idle compute unit, and the launch lasts as long as the
// longest chain in it: everything is asked for in one trip to memory, eight threads add a class's row and column, and the sums in
// a fixed order read their terms from LDS all at once.  90 x 160 cells, 19 classes: the launch that closes a call 5.6 -> 5.0 us, a scored
// frame 64.9 -> 63.3.  (Row and column added by one thread per class, and the mean by one thread that asked for a class at a time,
// were some 4000 cycles.)
template <bool EE, int NT = 256>
__device__ void finish_block(const FinishArgs& f, int block, int head)
{
    static_assert(NT >= 256 && 1024 % NT == 0, "eight threads per class; whole trips over the counts");
    __shared__ double part[256];
    __shared__ unsigned long long cl[32 * 32];
    __shared__ __attribute__((aligned(16))) double iou[32];
    __shared__ int present[32];
    const int tid = threadIdx.x;
    if (block == f.fph) {
        const unsigned long long nv = f.n_valid[head];
        if (tid < 256) {
            // a thread's contiguous run in ascending order, eight loads in flight (those beyond the run repeat its last)
            double acc = 0.0;
            const int per = (f.pph + 255) / 256;
            const float* lp = f.loss_part + (size_t)head * f.pph;
            const int end = min(f.pph, (tid + 1) * per);
            for (int i = tid * per; i < end; i += 8) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = lp[min(i + e, end - 1)];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (i + e < end) acc += (double)v[e];
            }
            part[tid] = acc;
        }
        __syncthreads();
        if (tid >= 64) return;
        double sum = (part[tid] + part[tid + 128]) + (part[tid + 64] + part[tid + 192]);
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) sum += __shfl_down(sum, s, 64);
        if (tid == 0 && f.loss_out) f.loss_out[head] = nv ? (float)(sum / (double)nv) : 0.f;
        return;
    }
    block += head * f.fph;      // the frame
    const int C = f.C;
    unsigned long long* cf = f.conf + (size_t)block * C * C;
    constexpr int TRIPS = 1024 / NT;
    unsigned long long v[TRIPS];
#pragma unroll
    for (int k = 0; k < TRIPS; ++k) v[k] = cf[min(tid + k * NT, C * C - 1)];
#pragma unroll
    for (int k = 0; k < TRIPS; ++k)
        if (tid + k * NT < C * C) cl[tid + k * NT] = v[k];
    __syncthreads();
    // (every thread has its counts by now: cleared for the next pass)
#pragma unroll
    for (int k = 0; k < TRIPS; ++k) {
        const int i = tid + k * NT;
        if (i >= C * C) continue;
        if (f.conf_out) f.conf_out[(size_t)block * C * C + i] = (long long)v[k];
        cf[i] = 0ull;
    }
    // IoU_c = conf[c][c] / (row_c + col_c - conf[c][c]) for classes with row_c > 0, added in
    // ascending c in float64 (the others add zero), divided by their number; 0 when no class is present
    if (tid < 256) {
        const int c = tid >> 3;
        unsigned long long row = 0, col = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int k = (tid & 7) + 8 * m;
            if (c < C && k < C) { row += cl[c * C + k]; col += cl[k * C + c]; }
        }
#pragma unroll
        for (int d = 4; d; d >>= 1) { row += __shfl_xor(row, d, 64); col += __shfl_xor(col, d, 64); }
        if ((tid & 7) == 0) {
            const unsigned long long inter = c < C ? cl[c * C + c] : 0;
            present[c] = row != 0;
            iou[c] = row ? (double)inter / (double)(row + col - inter) : 0.0;
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    const int cnt = __popcll(__ballot(tid < 32 && present[tid & 31]));
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 32; q += 8) {
        if (q >= C) break;
        double t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = iou[q + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += t[e];
    }
    if (tid == 0) {
        const double m = cnt ? sum / cnt : 0.0;
        if (f.miou_a) f.miou_a[block] = m;
        if (f.miou_b) f.miou_b[block] = m;
        if (EE && f.miou_c) {
            // host memory: the value, then the pass's token as a release at system scope, so a host
            // that sees the token also sees the value
            f.miou_c[block] = m;
            if (f.token_c) __hip_atomic_store(&f.token_c[block], f.token, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

}  // namespace st
