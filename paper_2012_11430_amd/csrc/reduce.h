// Deterministic reduction of per-workgroup partial rows in a separate launch.
//
// The fused kernels store one row of `tot` pairs per workgroup. A finishing
// launch (visibility of the rows is given by the kernel boundary) sums them:
// a workgroup owns 16 consecutive outputs; thread (row lane rl, output o) sums
// rows rl, rl + lanes, ... in order, with up to 16 loads in flight, then the row
// lanes of each output are added in a fixed order (FP64). The result does not
// depend on scheduling.
//
// What bounds it is the number of loads a thread waits for one after another: 64 row
// lanes per workgroup instead of 16 took 884 rows of 800 outputs from 5.8 to 4.7 us and
// 1022 rows of 2700 from 9.0 to 7.8; up to 512 rows (two rounds of loads) the two are
// equal or the small workgroup is faster (256 rows of 800: 2.3 to 3.9 against 3.9).
#pragma once

#include "common.h"

namespace prony {

constexpr int kFinishThreads = 256;                     // few rows
constexpr int kFinishThreadsMany = 1024;
constexpr int kFinishMany = 768;                        // rows from which these are taken
constexpr int kFinishOuts = 16;                         // outputs per workgroup

inline int finish_threads(int rows) { return rows >= kFinishMany ? kFinishThreadsMany : kFinishThreads; }

// Sum over `nrows` rows of column o0 + (tid % 16) of the row-major array `rows`
// (row length tot). Calls emit(o, re, im) once per owned output (o < tot).
template <int Threads = kFinishThreads, typename P2, typename Emit>
__device__ __forceinline__ void finish_rows(const P2* __restrict__ rows, int nrows, int tot, int o0, Emit emit) {
    constexpr int kLanes = Threads / kFinishOuts, kParts = kLanes / 16;
    __shared__ double2 red[kLanes][kFinishOuts];
    const int tid = threadIdx.x;
    const int oi = tid % kFinishOuts, rl = tid / kFinishOuts;
    const int o = o0 + oi;
    double re = 0.0, im = 0.0;
    if (o < tot) {
        constexpr int kBatch = 16;
        for (int r0 = rl; r0 < nrows; r0 += kBatch * kLanes) {
            P2 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int r = r0 + u * kLanes;
                if (r < nrows) v[u] = rows[(size_t)r * tot + o];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (r0 + u * kLanes < nrows) {
                    re += (double)v[u].x;
                    im += (double)v[u].y;
                }
            }
        }
    }
    red[rl][oi] = make_double2(re, im);
    __syncthreads();
    // runs of 16 lanes, then the runs
    if (kParts > 1) {
        re = im = 0.0;
        if (rl < kParts)
            for (int k = 0; k < 16; ++k) {
                re += red[16 * rl + k][oi].x;
                im += red[16 * rl + k][oi].y;
            }
        __syncthreads();
        if (rl < kParts) red[rl][oi] = make_double2(re, im);
        __syncthreads();
    }
    if (rl == 0 && o < tot) {
        re = 0.0;
        im = 0.0;
        for (int k = 0; k < (kParts > 1 ? kParts : 16); ++k) {
            re += red[k][oi].x;
            im += red[k][oi].y;
        }
        emit(o, re, im);
    }
}

}  // namespace prony
