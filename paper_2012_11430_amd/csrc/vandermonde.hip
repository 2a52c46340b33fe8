// Vandermonde products of the coefficient least-squares step (Sec. 1, eq. ls_probl;
// Algorithm 1, last line): A^T[k,j] = prod_l z_j(l)^{k_l}, gram = (A^T)^* A^T and
// rhs = (A^T)^* f_I, reduced over k in I_n. FP64 throughout.
//
// coeffs_tiles: a workgroup evaluates rows of A^T into LDS 16 at a time
//               (integer powers by binary exponentiation), optionally writes
//               them out, and accumulates its part of the Gram matrix and
//               right-hand side.
// coeffs_finish: sums the parts in a fixed order (reduce.h).
// coeffs_box:    both in one launch without A^T: a sum over the box I_n of a product over
//                the axes is the product of the axes' sums.
#include <algorithm>

#include "common.h"
#include "reduce.h"

namespace prony {
namespace {

constexpr int kRows = 16;        // rows of A^T per chunk
constexpr int kThreads = 256;
constexpr int kMaxM = 64;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ double2 cpow_int(double2 z, int e) {
    double2 r = make_double2(1.0, 0.0);
    double2 b = z;
    while (e) {
        if (e & 1) r = cmul(r, b);
        e >>= 1;
        if (e) b = cmul(b, b);
    }
    return r;
}

constexpr int kEntries = (kMaxM * kMaxM + kMaxM + kThreads - 1) / kThreads;

// Entry e of (A^T)^* [A^T | f_I]: the first m*m are the Gram matrix, the last m the rhs.
__device__ __forceinline__ void emit_gram(int m, double2* __restrict__ gram, double2* __restrict__ rhs, int e,
                                          double re, double im) {
    if (e < m * m)
        gram[e] = make_double2(re, im);
    else
        rhs[e - m * m] = make_double2(re, im);
}

// One workgroup takes `chunks` consecutive 16-row chunks of I_n. Per chunk the
// rows of A^T are evaluated into LDS, then every thread accumulates its fixed
// entries of (A^T)^* [A^T | f_I] over the chunk in FP64 registers. The
// workgroup's sums are stored as one row of partials; coeffs_finish adds the
// rows in workgroup order (bitwise reproducible) and writes gram and rhs.
__global__ __launch_bounds__(kThreads) void coeffs_tiles(int d, int n, int N, int m, int chunks,
                                                         const double2* __restrict__ z,
                                                         const double2* __restrict__ f, double2* __restrict__ at_out,
                                                         double2* __restrict__ part) {
    __shared__ double2 sz[kMaxM * 3];
    __shared__ double2 sa[kRows * kMaxM];
    __shared__ double2 sf[kRows];
    const int tid = threadIdx.x;
    const int tot = m * m + m;
    for (int i = tid; i < m * d; i += kThreads) sz[i] = z[i];
    const int c0 = grid_center(d, n);
    const int P = n + 1;
    double re[kEntries], im[kEntries];
#pragma unroll
    for (int u = 0; u < kEntries; ++u) re[u] = im[u] = 0.0;

    const int nchunks = (N + kRows - 1) / kRows;
    const int c_end = min((blockIdx.x + 1) * chunks, nchunks);
    for (int ch = blockIdx.x * chunks; ch < c_end; ++ch) {
        const int k0 = ch * kRows;
        __syncthreads();
        for (int r = tid; r < kRows; r += kThreads) {
            const int k = k0 + r;
            sf[r] = k < N ? f[grid_offset_of_index(k, d, n) + c0] : make_double2(0.0, 0.0);
        }
        for (int e = tid; e < kRows * m; e += kThreads) {
            const int r = e / m, j = e - (e / m) * m;
            const int k = k0 + r;
            double2 a = make_double2(0.0, 0.0);
            if (k < N) {
                a = make_double2(1.0, 0.0);
                int rem = k;
                for (int l = d - 1; l >= 0; --l) {
                    const int q = rem / P;
                    a = cmul(a, cpow_int(sz[j * d + l], rem - q * P));
                    rem = q;
                }
                if (at_out) at_out[(size_t)k * m + j] = a;
            }
            sa[r * kMaxM + j] = a;
        }
        __syncthreads();
        const int rows = min(kRows, N - k0);
#pragma unroll
        for (int u = 0; u < kEntries; ++u) {
            const int e = tid + u * kThreads;
            if (e < tot) {
                const int i = e < m * m ? e / m : e - m * m;
                const int j = e < m * m ? e - (e / m) * m : -1;
                for (int r = 0; r < rows; ++r) {
                    const double2 ai = sa[r * kMaxM + i];
                    const double2 b = j >= 0 ? sa[r * kMaxM + j] : sf[r];
                    // conj(ai) * b
                    re[u] = fma(ai.x, b.x, fma(ai.y, b.y, re[u]));
                    im[u] = fma(ai.x, b.y, fma(-ai.y, b.x, im[u]));
                }
            }
        }
    }
    double2* out = part + (size_t)blockIdx.x * tot;
#pragma unroll
    for (int u = 0; u < kEntries; ++u) {
        const int e = tid + u * kThreads;
        if (e < tot) out[e] = make_double2(re[u], im[u]);
    }
}

// Sum of the workgroup parts (reduce.h) into gram and rhs.
__global__ __launch_bounds__(kFinishThreads) void coeffs_finish(int m, int rows, const double2* __restrict__ part,
                                                                double2* __restrict__ gram,
                                                                double2* __restrict__ rhs) {
    finish_rows(part, rows, m * m + m, blockIdx.x * kFinishOuts,
                [&](int e, double re, double im) { emit_gram(m, gram, rhs, e, re, im); });
}

// gram[i, j] = sum over k in I_n of prod_l conj(z_i(l)^k_l) z_j(l)^k_l
//            = prod_l sum_{k <= n} conj(z_i(l)^k) z_j(l)^k,
// m^2 d (n + 1) products instead of m^2 (n + 1)^d, so that a row of the Gram matrix is one
// workgroup's work and an entry of the right-hand side another's (workgroups m + i).
// Powers are formed as in coeffs_tiles, by binary exponentiation every kStep and by
// products in between. What is left is latency, one pass of loads, powers and sums:
// d=2 n=63 m=20 7.2 to 9.6 us against 8.9 + 3.5 us of the two launches above, which stay for
// A^T itself and past the sizes of box_fits. All loads are requested before the powers of z_i.
constexpr int kStep = 8, kLanes = 8;         // powers per run; lanes of one sum
constexpr int kBoxThreads = 512;

__global__ __launch_bounds__(kBoxThreads) void coeffs_box(int d, int n, int N, int m, const double2* __restrict__ z,
                                                          const double2* __restrict__ f, double2* __restrict__ gram,
                                                          double2* __restrict__ rhs) {
    extern __shared__ __align__(16) unsigned char smem[];
    double2* pw = reinterpret_cast<double2*>(smem);      // z_i(l)^k at l E + k
    __shared__ double2 axis[kMaxM * 3];
    __shared__ double2 waves[kBoxThreads / 64];
    const int tid = threadIdx.x, E = n + 1;
    const bool row = blockIdx.x < (unsigned)m;
    const int i = row ? blockIdx.x : blockIdx.x - m;
    const int runs = (E + kStep - 1) / kStep;
    constexpr int kIn = 8;
    const int c0 = grid_center(d, n), lane = tid % kLanes;
    double2 v[kIn], zl = make_double2(0.0, 0.0);
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kIn; ++u) {
            const int k = k0 + u * kBoxThreads;
            v[u] = k < N ? f[grid_offset_of_index(k, d, n) + c0] : make_double2(0.0, 0.0);
        }
    };
    if (row) {
        if (tid / kLanes < m * d) zl = z[tid / kLanes];
    } else {
        load(tid);
    }
    for (int e = tid; e < d * runs; e += kBoxThreads) {
        const int l = e / runs, k0 = (e - l * runs) * kStep;
        const double2 zi = z[i * d + l];
        double2 p = cpow_int(zi, k0);
        for (int k = k0; k < min(k0 + kStep, E); ++k) {
            pw[l * E + k] = p;
            p = cmul(p, zi);
        }
    }
    if (row) {
        for (int e0 = 0; e0 < m * d; e0 += kBoxThreads / kLanes) {
            const int e = e0 + tid / kLanes, l = e % d;
            double2 p = cpow_int(zl, lane * kStep);
            if (e0 == 0) __syncthreads();
            double re = 0.0, im = 0.0;
            for (int r = lane; r < runs; r += kLanes) {
                if (r > lane) p = cpow_int(zl, r * kStep);
                for (int k = r * kStep; k < min((r + 1) * kStep, E); ++k) {
                    const double2 a = pw[l * E + k];
                    re = fma(a.x, p.x, fma(a.y, p.y, re));
                    im = fma(a.x, p.y, fma(-a.y, p.x, im));
                    p = cmul(p, zl);
                }
            }
#pragma unroll
            for (int x = 1; x < kLanes; x *= 2) {
                re += __shfl_xor(re, x);
                im += __shfl_xor(im, x);
            }
            if (lane == 0 && e < m * d) axis[e] = make_double2(re, im);
            if (e + kBoxThreads / kLanes < m * d) zl = z[e + kBoxThreads / kLanes];
        }
        __syncthreads();
        for (int j = tid; j < m; j += kBoxThreads) {
            double2 s = axis[j * d];
            for (int l = 1; l < d; ++l) s = cmul(s, axis[j * d + l]);
            gram[(size_t)i * m + j] = s;
        }
        return;
    }
    __syncthreads();
    double re = 0.0, im = 0.0;
    for (int k0 = tid; k0 < N; k0 += kIn * kBoxThreads) {
        if (k0 > tid) load(k0);
#pragma unroll
        for (int u = 0; u < kIn; ++u) {
            const int k = k0 + u * kBoxThreads;
            if (k >= N) break;
            int rem = k / E;
            double2 a = pw[(d - 1) * E + k - rem * E];
            for (int l = d - 2; l >= 0; --l) {
                const int q = rem / E;
                a = cmul(a, pw[l * E + rem - q * E]);
                rem = q;
            }
            re = fma(a.x, v[u].x, fma(a.y, v[u].y, re));
            im = fma(a.x, v[u].y, fma(-a.y, v[u].x, im));
        }
    }
#pragma unroll
    for (int x = 1; x < 64; x *= 2) {
        re += __shfl_xor(re, x);
        im += __shfl_xor(im, x);
    }
    if (tid % 64 == 0) waves[tid / 64] = make_double2(re, im);
    __syncthreads();
    if (tid == 0) {
        double2 s = waves[0];
        for (int w = 1; w < kBoxThreads / 64; ++w) {
            s.x += waves[w].x;
            s.y += waves[w].y;
        }
        rhs[i] = s;
    }
}

// The box's time does not depend on m but grows with the line (a lane takes every 8th run of
// powers one after another: 25.5 us at d = 1, n = 1023) and with the samples that one workgroup
// reads; the tiles' grows with m past 16. Calls in us, box / tiles: d=1 n=447 m=20 12.2 / 12.3,
// n=511 13.6 / 12.6, n=511 m=40 13.7 / 14.6, n=767 m=64 19.9 / 24.5; d=2 n=111 m=12 14.7 / 18.0,
// n=127 18.4 / 18.4; d=3 n=20 m=12 15.6 / 15.6, n=22 19.3 / 15.9, n=24 m=20 24.1 / 27.6.
bool box_fits(int d, int n, int64_t N, int m) {
    const int line = m <= 32 ? 448 : m <= 48 ? 544 : 896;
    const int rows = m > 16 ? 16384 : d == 3 ? 9600 : 14400;
    return n + 1 <= line && N <= rows;
}

constexpr int kMaxWorkgroups = 256;   // one 16-row chunk each for N <= 4096

}  // namespace

size_t coeffs_workspace_bytes(int d, int n, int m) {
    (void)d;
    (void)n;
    return align_up((size_t)kMaxWorkgroups * (m * m + m) * sizeof(double2), 256);
}

}  // namespace prony

using namespace prony;

extern "C" prony_status_t prony_coeffs(prony_handle_t h, int d, int n, int m, const double* z, const double* f,
                                       double* gram, double* rhs, double* AT_out) {
    if (!h) return PRONY_EINVAL;
    prony_status_t st = check_dn(h, d, n);
    if (st != PRONY_OK) return st;
    const int64_t N = ipow(n + 1, d);
    if (m < 1 || m > N) return fail(h, PRONY_EINVAL, "prony_coeffs: m must be in 1..N");
    if (m > kMaxM) return fail(h, PRONY_ENOTSUP, "prony_coeffs: m > 64 is not supported");
    if (!z || !f || !gram || !rhs) return fail(h, PRONY_EINVAL, "prony_coeffs: null pointer");
    if (h->device < 0) return fail(h, PRONY_ENODEV, "validation-only handle has no device");
    DeviceGuard g(h->device);
    if (!g.ok) return fail(h, PRONY_EHIP, "hipSetDevice failed");
    if ((st = ensure_workspace(h, coeffs_workspace_bytes(d, n, m))) != PRONY_OK) return st;
    if (!AT_out && box_fits(d, n, N, m)) {
        {
            ProfileScope prof(h, "coeffs_tiles");
            coeffs_box<<<2 * m, kBoxThreads, 16 * (size_t)d * (n + 1), h->stream>>>(
                d, n, (int)N, m, reinterpret_cast<const double2*>(z), reinterpret_cast<const double2*>(f),
                reinterpret_cast<double2*>(gram), reinterpret_cast<double2*>(rhs));
        }
        return check_launch(h, "coeffs_box");
    }
    const int nchunks = (int)((N + kRows - 1) / kRows);
    const int chunks = (nchunks + kMaxWorkgroups - 1) / kMaxWorkgroups;
    const int wgs = (nchunks + chunks - 1) / chunks;
    double2* part = static_cast<double2*>(h->ws);
    {
        ProfileScope prof(h, "coeffs_tiles");
        coeffs_tiles<<<wgs, kThreads, 0, h->stream>>>(d, n, (int)N, m, chunks, reinterpret_cast<const double2*>(z),
                                                      reinterpret_cast<const double2*>(f),
                                                      reinterpret_cast<double2*>(AT_out), part);
    }
    if ((st = check_launch(h, "coeffs_tiles")) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "coeffs_finish");
        const int tot = m * m + m;
        coeffs_finish<<<(tot + kFinishOuts - 1) / kFinishOuts, kFinishThreads, 0, h->stream>>>(
            m, wgs, part, reinterpret_cast<double2*>(gram), reinterpret_cast<double2*>(rhs));
    }
    return check_launch(h, "coeffs_finish");
}
