// FP64 S-build in line-spectral form.
//
// S_l = U_l^* T_row V with T_row[k', h] = f(k' - h) (the row-extended form of
// pencil.hip). Along the axes 2..d both index sets lie in an embedding of
// L = 2(n+1) points on which k' - h in {-n..n+1} is a circular difference, so a DFT
// of length L along these axes (x~(w) = sum_k x(k) e^{-2 pi i <w,k>/L}) turns T_row
// into F = L^(d-1) independent one-dimensional Toeplitz matrices along axis 1,
//     Y_w[k1'] = sum_h1 f~_w(k1' - h1) V~_w[h1],
// and, since a shift of U by e_l (l >= 2) is the phase e^{-2 pi i w_l / L},
//     U_l^* T_row V = 1/F sum_w e^{2 pi i w_l / L} sum_k1 U~_w[k1]^* Y_w[k1]   (l >= 2),
//     U_1^* T_row V = 1/F sum_w sum_k1 U~_w[k1]^* Y_w[k1 + 1].
// Per instance this takes 8 (n+2)(n+1) m L^(d-1) operations for the products instead
// of 8 (n+2)^d (n+1)^d m, plus the transforms of U, V and f, for results of the same
// precision: every sum is FP64, and the lengths of the sums fall from (n+1)^d to
// (d-1)(n+1) + (n+1). d = 1: k = k1 P + k2 is folded into K1 lines of P points, which
// makes T a two-level Toeplitz matrix with f2(p1, p2) = f(p1 P + p2); S_1 is then the
// phase form along the second level.
//
//   spectral_forward  DFTs of U, V and f as real contractions with the cosine and sine
//                     tables on the FP64 matrix cores: frequency w and its mirror L - w
//                     share both sums, x~(w), x~(L - w) = C -+ i S;
//   spectral_gram     per frequency the Toeplitz product (window of f~_w in LDS) and the
//                     two Gram products, chained in registers: the 16x16 FP64 result
//                     layout (lane group g, element r: row g + 4 r) is the second
//                     operand's layout of K step r, so Y_w never leaves the registers;
//   spectral_finish   fixed-order sum of the groups' partials, Sigma^{-1}.
#include <algorithm>
#include <cmath>
#include <new>
#include <type_traits>
#include <vector>

#include "mfma.h"
#include "reduce.h"
#include "spectral.h"

namespace prony {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kCols = 8;            // complex columns of one 16-column MFMA block
using M = Mfma<double>;
using acc_t = M::acc_t;

// Table in LDS of cos and sin of 2 pi j / L, j < L, one entry skipped after every 16 (all
// banks): the rows of a block read it at strides 4 s + g, which without the gaps fall
// into few banks where L is a multiple of 16.
__host__ __device__ inline int root_slot(int j) { return j + (j >> 4); }
__host__ __device__ inline size_t roots_bytes(int L) { return 16 * (size_t)(root_slot(L - 1) + 1); }
__device__ __forceinline__ void fill_roots(double2* tab, int L) {
    for (int j = threadIdx.x; j < L; j += kThreads) {
        double s, c;
        sincospi(2.0 * j / L, &s, &c);
        tab[root_slot(j)] = make_double2(c, s);
    }
}

// LDS rows of one staged line block (whole groups of K steps) and doubles per row of
// the planes between the two transforms of d = 3 (rows 128 bytes apart modulo 256:
// the rows of two lane groups fall into different banks).
__host__ __device__ inline int line_rows(int K) { return (K + 15) & ~15; }
__host__ __device__ inline int plane_stride(int pairs, int nq) { return ((4 * pairs * nq + 31) & ~31) + 16; }
__host__ __device__ inline int inverse_stride(int rows, int nq) { return ((2 * rows * nq + 31) & ~31) + 16; }

// Offset in f of the sample (line t, point j of the embedded axis), -1 where there is
// none (the products with T use the samples up to n only). Point j stands for
// p2 = j (j <= P) or j - L.
__device__ __forceinline__ int sample_offset(const SpecPlan& P, int t, int j) {
    const int p1 = t - (P.K1 - 1), p2 = j <= P.P ? j : j - P.L;
    if (P.d == 2) return p1 <= P.pmax && p2 <= P.pmax ? (p1 + P.n) * P.L + p2 + P.n : -1;
    const int p = p1 * P.P + p2;
    return p >= -P.n && p <= P.pmax ? p + P.n : -1;
}

// Forward transforms run on 16-row blocks of 8 frequency pairs: row i < 8 of block pb
// is the cosine row of w = w0 + 8 pb + i, row 8 + i its sine row, so that a lane holds
// C = sum x cos (elements 0, 1) and S = sum x sin (elements 2, 3) of the pairs
// g and g + 4 of the block. Frequency 0 has no sine row: its slot holds the signs
// (-1)^j of frequency P.
constexpr int kPairs = 8;

// First index and step of a walk x g, x (g + 4), x (g + 8), ... modulo L, g < 4, x < L / 2
// (rows past the last are clamped to it; they are not stored).
__device__ __forceinline__ void walk_start(int x, int g, int L, int& idx, int& step) {
    x = min(x, L / 2 - 1);
    idx = x * g;
    if (idx >= L) idx -= L;
    step = 4 * x;
    if (step >= L) step -= L;
}

// Table walk of a lane's row: its factor at j = 4 s + g for s = 0, 1, ...
struct RowWalk {
    int idx, step, L, part;
    double alt;
    bool zero_sine;
    __device__ __forceinline__ RowWalk(int w, bool sine, int g, int L_) {
        L = L_;
        walk_start(w, g, L, idx, step);
        part = sine ? 1 : 0;
        alt = g & 1 ? -1.0 : 1.0;
        zero_sine = sine && w == 0;
    }
    __device__ __forceinline__ double next(const double2* tab) {
        const double v = reinterpret_cast<const double*>(tab)[2 * root_slot(idx) + part];
        idx += step;
        if (idx >= L) idx -= L;
        return zero_sine ? alt : v;
    }
};

// x~(w) and x~(L - w) (one real column of a complex one, whose other component sits in
// the neighbouring lane): C -+ i S; for w = 0 the frequencies 0 and P.
__device__ __forceinline__ void pair_out(int w, bool odd, double C, double S, double scale, double& lo, double& hi) {
    const double x = swap_lane_pair(S), y = odd ? -x : x;
    lo = (w == 0 ? C : C + y) * scale;
    hi = (w == 0 ? S : C - y) * scale;
}

// Forward transform with one transformed axis (d <= 2): nbc blocks of 8 complex
// columns from block nb0. Columns of a factor: c = line * m + q; of the grid: the
// sample lines t. out[w * NC + c].
__device__ __forceinline__ void forward_lines(const SpecPlan& P, const double2* __restrict__ src, int64_t rs,
                                              int64_t cs, bool grid, double2* __restrict__ out, int nb0, int nbc,
                                              unsigned char* smem) {
    const int mc = grid ? 1 : P.m;
    const int NC = grid ? P.NP1 : P.K1 * P.m;
    const int K = grid ? P.L : P.P, KS = (K + 3) >> 2, J = line_rows(K);
    double2* tab = reinterpret_cast<double2*>(smem);
    double2* xs = tab + roots_bytes(P.L) / 16;                     // [block][j][8 columns]
    const int tid = threadIdx.x;
    // the inputs in tiles of 16 points x 8 columns per half workgroup, lanes along the
    // axis that is contiguous in memory, 8 loads in flight
    const bool jfast = grid || rs < cs;
    const int e = tid & 127, jl = jfast ? e & 15 : e >> 3, cc = jfast ? e >> 4 : e & 7;
    const int half = tid >> 7, per = (J / 16 + 1) / 2, turns = nbc * per;   // turns of both halves
    constexpr int kStage = 8;
    for (int base = 0; base < turns; base += kStage) {
        double2 v[kStage];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            v[u] = make_double2(0.0, 0.0);
            if (base + u < turns) {
                const int nb = (base + u) / per, j = 16 * (2 * (base + u - nb * per) + half) + jl;
                const int c = kCols * (nb0 + nb) + cc;
                if (c < NC && j < K) {
                    if (grid) {
                        const int o = sample_offset(P, c, j);
                        if (o >= 0) v[u] = src[o];
                    } else {
                        const int line = c / mc, q = c - line * mc, idx = line * P.P + j;
                        if (idx < P.N) v[u] = src[idx * rs + q * cs];
                    }
                }
            }
        }
        if (base == 0) fill_roots(tab, P.L);
#pragma unroll
        for (int u = 0; u < kStage; ++u)
            if (base + u < turns) {
                const int nb = (base + u) / per, j = 16 * (2 * (base + u - nb * per) + half) + jl;
                if (j < J) xs[(nb * J + j) * kCols + cc] = v[u];
            }
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, g = lane >> 4, col = lane & 15;
    const bool odd = lane & 1;
    const double scale = grid ? 1.0 / P.F : 1.0;
    // an item is one column block against two blocks of pairs, four K steps of
    // operands ahead
    constexpr int NP = 2, CH = 4;
    const int npi = (P.npb + NP - 1) / NP;
    for (int it = wave; it < nbc * npi; it += kWaves) {
        const int nb = it / npi, pb = (it - nb * npi) * NP;
        RowWalk row[NP] = {RowWalk(kPairs * pb + (col & 7), col >= 8, g, P.L),
                           RowWalk(kPairs * (pb + 1) + (col & 7), col >= 8, g, P.L)};
        const double* x = reinterpret_cast<const double*>(xs + (size_t)nb * J * kCols) + 16 * g + col;
        acc_t acc[NP];
        double a[2][CH][NP], b[2][CH];
        auto read = [&](int buf, int s) {       // rows past K are zero
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                b[buf][k] = x[64 * (s + k)];
#pragma unroll
                for (int i = 0; i < NP; ++i) a[buf][k][i] = row[i].next(tab);
            }
        };
        auto mma = [&](int buf, int s) {
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (s + k < KS)
#pragma unroll
                    for (int i = 0; i < NP; ++i) acc[i] = M::fma(a[buf][k][i], b[buf][k], acc[i]);
        };
#pragma unroll
        for (int i = 0; i < NP; ++i) acc[i] = acc_t{0, 0, 0, 0};
        read(0, 0);
        for (int s = 0; s < KS; s += 2 * CH) {
            if (s + CH < KS) read(1, s + CH);
            mma(0, s);
            if (s + 2 * CH < KS) read(0, s + 2 * CH);
            mma(1, s + CH);
        }
        const int c = kCols * (nb0 + nb) + (col >> 1);
        double* o = reinterpret_cast<double*>(out) + 2 * c + (col & 1);
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int w = kPairs * (pb + i) + g + 4 * r;
                double lo, hi;
                pair_out(w, odd, acc[i][r], acc[i][r + 2], scale, lo, hi);
                if (w < P.P && c < NC) {
                    o[(size_t)w * NC * 2] = lo;
                    o[(size_t)(w == 0 ? P.P : P.L - w) * NC * 2] = hi;
                }
            }
    }
}

// Forward transform with two transformed axes (d = 3): the plane (axes 2, 3) of line
// `line` and nq complex columns from column q0: axis 3 at the pairs split * wp ..
// (and their mirrors) into LDS, then axis 2. out[(w2 L + w3) * rowlen + line * mc + q].
__device__ __forceinline__ void forward_planes(const SpecPlan& P, const double2* __restrict__ src, int64_t rs,
                                               int64_t cs, bool grid, double2* __restrict__ out, int line, int q0,
                                               int nq, int split, unsigned char* smem) {
    const int mc = grid ? 1 : P.m;
    const size_t rowlen = grid ? P.NP1 : (size_t)P.K1 * P.m;
    const int J = grid ? P.L : P.P, KS = (J + 3) >> 2;
    const int w0 = split * P.wp, wn = min(P.wp, P.P - w0);
    double2* tab = reinterpret_cast<double2*>(smem);
    double* t1 = reinterpret_cast<double*>(tab + roots_bytes(P.L) / 16);      // [j2][2 u + side][q] complex
    const int ts = plane_stride(wn, nq);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, col = lane & 15;
    const bool odd = lane & 1, sine = col >= 8;
    const int jskip = P.pmax == P.n ? P.P : -1;      // the point p = n + 1 of an axis
    const double* in = reinterpret_cast<const double*>(src);
    // rows past J are zero (the K steps are whole)
    for (int i = tid; i < (4 * KS - J) * ts; i += kThreads) t1[(size_t)J * ts + i] = 0.0;

    // axis 3: columns c = j2 * nq + q in blocks of 8, NBI blocks per pass, so that one
    // read of the tables serves all, and kIn K steps of their loads in flight
    constexpr int NBI = 2, kIn = 6;
    const int nc1 = J * nq, nb1 = (nc1 + 7) >> 3, npb1 = (wn + kPairs - 1) / kPairs;
    const int items1 = (nb1 + NBI - 1) / NBI * npb1;
    const float rnq = 1.0f / nq;
    auto div_nq = [&](int c) { return (int)((c + 0.5f) * rnq); };     // c < 2^14: exact
    struct Item {
        bool live[NBI];          // columns of the plane
        int o1[NBI];             // their places in an LDS row
        const double* x[NBI];    // their first inputs, null where there are none
    };
    auto item_at = [&](int it, Item& I) {
        const int ng = it / npb1;
#pragma unroll
        for (int i = 0; i < NBI; ++i) {
            const int c = 8 * (ng * NBI + i) + (col >> 1);
            I.live[i] = it < items1 && c < nc1;
            const int j2 = div_nq(c), q = c - j2 * nq;
            I.o1[i] = j2 * ts + 2 * q + (col & 1);
            bool ok = I.live[i];
            int64_t base;
            if (grid) {
                const int p1 = line - (P.K1 - 1), p2 = j2 <= P.P ? j2 : j2 - P.L;
                ok = ok && p1 <= P.pmax && p2 <= P.pmax;
                base = 2 * ((int64_t)((p1 + P.n) * P.L + p2 + P.n) * P.L + P.n) + (col & 1);
            } else {
                base = 2 * ((int64_t)(line * P.P + j2) * P.P * rs + (q0 + q) * cs) + (col & 1);
            }
            I.x[i] = ok ? in + base : nullptr;
        }
    };
    auto load = [&](double (&b)[NBI][kIn], const Item& I, int s0) {
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const int j = 4 * (s0 + k) + g;
            const int64_t off = grid ? (int64_t)(j <= P.P ? j : j - P.L) * 2 : 2 * j * rs;
            const bool ok = j < J && (!grid || j != jskip);
#pragma unroll
            for (int i = 0; i < NBI; ++i) b[i][k] = I.x[i] && ok ? I.x[i][off] : 0.0;
        }
    };
    Item item;
    double b[NBI][kIn];
    item_at(wave, item);
    load(b, item, 0);
    fill_roots(tab, P.L);            // the first loads are in flight
    __syncthreads();
    for (int it = wave; it < items1; it += kWaves) {
        const int pb = it % npb1;
        acc_t acc[NBI];
#pragma unroll
        for (int i = 0; i < NBI; ++i) acc[i] = acc_t{0, 0, 0, 0};
        Item next;
        item_at(it + kWaves, next);
        RowWalk row(w0 + kPairs * pb + (col & 7), sine, g, P.L);
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            double a[kIn], bn[NBI][kIn];
            // the next K steps or the next item's first ones
            const bool more = s0 + kIn < KS;
            load(bn, more ? item : next, more ? s0 + kIn : 0);
#pragma unroll
            for (int k = 0; k < kIn; ++k) a[k] = row.next(tab);
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                if (s0 + k < KS)
#pragma unroll
                    for (int i = 0; i < NBI; ++i) acc[i] = M::fma(a[k], b[i][k], acc[i]);
#pragma unroll
            for (int i = 0; i < NBI; ++i)
#pragma unroll
                for (int k = 0; k < kIn; ++k) b[i][k] = bn[i][k];
        }
#pragma unroll
        for (int i = 0; i < NBI; ++i)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int u = kPairs * pb + g + 4 * r;
                double lo, hi;
                pair_out(w0 + u, odd, acc[i][r], acc[i][r + 2], 1.0, lo, hi);
                if (item.live[i] && u < wn) {
                    t1[item.o1[i] + 4 * u * nq] = lo;
                    t1[item.o1[i] + (4 * u + 2) * nq] = hi;
                }
            }
        item = next;
    }
    __syncthreads();

    // axis 2: columns c = (2 u + side) * nq + q of the LDS rows j2
    constexpr int NB2 = 4, CH = 3;
    const int nc2 = 2 * wn * nq, nb2 = (nc2 + 7) >> 3;
    const int ng2 = (nb2 + NB2 - 1) / NB2;
    const double scale = grid ? 1.0 / P.F : 1.0;
    for (int it = wave; it < ng2 * P.npb; it += kWaves) {
        const int ng = it / P.npb, pb = it - ng * P.npb;
        RowWalk row(kPairs * pb + (col & 7), sine, g, P.L);
        acc_t acc[NB2];
        const double* x[NB2];
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
            acc[i] = acc_t{0, 0, 0, 0};
            // columns past the last read the last block again and are not stored
            x[i] = t1 + g * ts + 16 * min(ng * NB2 + i, nb2 - 1) + col;
        }
        double a[2][CH], b[2][CH][NB2];
        auto read = [&](int buf, int s) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                a[buf][k] = row.next(tab);
#pragma unroll
                for (int i = 0; i < NB2; ++i) b[buf][k][i] = x[i][4 * min(s + k, KS - 1) * ts];
            }
        };
        auto mma = [&](int buf, int s) {
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (s + k < KS)
#pragma unroll
                    for (int i = 0; i < NB2; ++i) acc[i] = M::fma(a[buf][k], b[buf][k][i], acc[i]);
        };
        read(0, 0);
        for (int s = 0; s < KS; s += 2 * CH) {
            if (s + CH < KS) read(1, s + CH);
            mma(0, s);
            if (s + 2 * CH < KS) read(0, s + 2 * CH);
            mma(1, s + CH);
        }
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
            const int c = 8 * (ng * NB2 + i) + (col >> 1);
            const int wl = div_nq(c), q = c - wl * nq, w3p = w0 + (wl >> 1);
            const int w3 = wl & 1 ? (w3p == 0 ? P.P : P.L - w3p) : w3p;
            double* o = reinterpret_cast<double*>(out) + 2 * ((size_t)w3 * rowlen + (size_t)line * mc + q0 + q) + (col & 1);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int w2 = kPairs * pb + g + 4 * r;
                double lo, hi;
                pair_out(w2, odd, acc[i][r], acc[i][r + 2], scale, lo, hi);
                if (w2 < P.P && c < nc2) {
                    o[(size_t)w2 * P.L * rowlen * 2] = lo;
                    o[(size_t)(w2 == 0 ? P.P : P.L - w2) * P.L * rowlen * 2] = hi;
                }
            }
        }
    }
}

// Workgroup `id` of an instance's forward transforms: the sample grid's first (they
// are the longest), then V's and U's.
__device__ __forceinline__ void forward_body(const SpecPlan& P, const SpecPtrs& p, int id, unsigned char* smem) {
    const bool grid = id < P.wgs_f;
    const bool second = id >= P.wgs_f + P.wgs_x;
    if (id == 0)    // the phases of the Gram products
        for (int j = threadIdx.x; j < P.L; j += kThreads) {
            double sn, cn;
            sincospi(2.0 * j / P.L, &sn, &cn);
            p.roots[j] = make_double2(cn, sn);
        }
    const int x = grid ? id : id - P.wgs_f - (second ? P.wgs_x : 0);
    const double2* src = grid ? p.f : second ? p.U : p.V;
    const int64_t rs = second ? p.u_rs : p.v_rs, cs = second ? p.u_cs : p.v_cs;
    double2* out = grid ? p.ft : second ? p.ut : p.vt;
    if (P.d == 3) {
        const int per = grid ? 1 : (P.m + P.nq - 1) / P.nq;   // column blocks of a line
        const int split = x % P.splits, rest = x / P.splits;
        const int qb = rest % per, line = rest / per;
        forward_planes(P, src, rs, cs, grid, out, line, qb * P.nq, grid ? 1 : min(P.nq, P.m - qb * P.nq), split, smem);
    } else {
        const int nbw = grid ? P.nbwf : P.nbw;
        const int nblk = ((grid ? P.NP1 : P.K1 * P.m) + kCols - 1) / kCols;
        forward_lines(P, src, rs, cs, grid, out, x * nbw, min(nbw, nblk - x * nbw), smem);
    }
}

__global__ __launch_bounds__(kThreads) void spectral_forward_kernel(SpecPlan P, SpecPtrs p, int first) {
    extern __shared__ __align__(16) unsigned char smem[];
    forward_body(P, p, first + blockIdx.x, smem);
}

// A buffer of `bytes` bytes at `p` (wave-uniform): loads at byte offsets outside it,
// negative ones included, return zero. The offset kOutside stays outside when a
// buffer's length is added.
constexpr int kOutside = (int)0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const double2* p, int bytes) {
    constexpr int kRaw32 = 0x00020000;   // untyped 32-bit data, no swizzle
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double2*>(p), 0, bytes, kRaw32);
}
__device__ __forceinline__ double2 buffer_load(__amdgpu_buffer_rsrc_t b, int offset) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    typedef double d2 __attribute__((ext_vector_type(2)));
    const u4 v = __builtin_amdgcn_raw_buffer_load_b128(b, offset, 0, 0);
    const d2 d = __builtin_bit_cast(d2, v);
    return make_double2(d.x, d.y);
}

// Largest number of lines (a wave's window of f~_w is held in four registers per lane
// between its load and its LDS store: 16 + 4 KS - 1 <= 256 entries).
constexpr int kMaxLines = 240;
__host__ __device__ inline size_t window_bytes(int K1) { return 16 * (size_t)(16 + ((K1 + 3) & ~3)); }

// Rows r0 .. r0 + 15 of Y_w = T_w V~_w over the K steps s0 .. s1 - 1 (h1 = 4 s .. 4 s + 3)
// in the three-product form; lane (g, col) gets the rows r0 + g + 4 r, r < 4, of V's
// column col (at byte voff + h1 * 16 m of V~_w). adjoint: T_w^* instead of T_w, i.e.
// conj(f~_w(-p)) for f~_w(p). `between` runs after the first loads are requested.
template <int CH, typename Between>
__device__ __forceinline__ void toeplitz_rows(const SpecPlan& P, const SpecPtrs& p, int w, int r0, int s0, int s1,
                                              int voff, bool adjoint, double2* win, double (&yr)[4], double (&yi)[4],
                                              Between between) {
    const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
    const int row_bytes = 16 * P.m, K1 = P.K1;
    constexpr int NW = 4;
    const auto ft = buffer_of(p.ft + (size_t)w * P.NP1, 16 * P.NP1);
    const auto vt = buffer_of(p.vt + (size_t)w * K1 * P.m, K1 * row_bytes);
    // window entry x: row r0 + i, column h with x = i + 4 s1 - 1 - h
    const int t0 = r0 + K1 - 4 * s1, cnt = 15 + 4 * (s1 - s0);
    double2 wr[NW], va[CH], vb[CH];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const int t = t0 + lane + 64 * k;
        wr[k] = buffer_load(ft, 16 * (adjoint ? 2 * (K1 - 1) - t : t));
    }
    auto load_v = [&](double2 (&v)[CH], int s) {
#pragma unroll
        for (int k = 0; k < CH; ++k) v[k] = buffer_load(vt, voff + 4 * (s + k) * row_bytes);
    };
    load_v(va, s0);
    load_v(vb, s0 + CH);
    between();
#pragma unroll
    for (int k = 0; k < NW; ++k)
        if (64 * k < cnt && lane + 64 * k < cnt)
            win[lane + 64 * k] = adjoint ? make_double2(wr[k].x, -wr[k].y) : wr[k];
    __builtin_amdgcn_wave_barrier();
    acc_t y1 = {0, 0, 0, 0}, y2 = {0, 0, 0, 0}, y3 = {0, 0, 0, 0};
    const double2* wl = win + col + 4 * s1 - 1 - g;
    auto mma = [&](const double2 (&v)[CH], int s) {
#pragma unroll
        for (int k = 0; k < CH; ++k)
            if (s + k < s1) {
                const double2 a = wl[-4 * (s + k)];
                y1 = M::fma(a.x, v[k].x, y1);
                y2 = M::fma(a.y, v[k].y, y2);
                y3 = M::fma(a.x + a.y, v[k].x + v[k].y, y3);
            }
    };
    for (int s = s0; s < s1; s += 2 * CH) {
        mma(va, s);
        if (s + 2 * CH < s1) load_v(va, s + 2 * CH);
        mma(vb, s + CH);
        if (s + 3 * CH < s1) load_v(vb, s + 3 * CH);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        yr[r] = y1[r] - y2[r];
        yi[r] = y3[r] - y1[r] - y2[r];
    }
}

// Frequencies wa .. wb - 1 of group grp; with d = 3 they share the frequency of axis 2.
__device__ __forceinline__ void group_range(const SpecPlan& P, int grp, int& wa, int& wb) {
    const int gp = P.gparts, n = P.d == 3 ? P.L : P.F;
    const int o = grp / gp, k = grp - o * gp;
    wa = o * n + n * k / gp;
    wb = o * n + n * (k + 1) / gp;
}

// Weighted Gram products of the frequencies of group grp with the columns
// 16 qb .. 16 qb + 15 of V. Per 16-row block of rows k1': the Toeplitz product in the
// three-product form, then the Gram products with the stacked rows
// [U~_w[k1] | U~_w[k1 - 1]] (d >= 2; the second m rows give S_1): NMB blocks of 16, of
// which the first NM0 hold rows of the first kind. NS = 1: their sum with the phase
// e^{2 pi i w_d / L}; NS = 2: the plain sum and the one with that phase (d = 3: axis 2's
// phase is the group's, applied to the plain sum at the end). The shifted rows take the
// plain sum in either case. At most 256 registers, so that two workgroups share a CU and
// one's loads overlap the other's products. Requesting the next row block's operands
// before the Gram products, or running the full and partial block of a frequency
// together on shared V operands, took the kernel past that and lost more to spills
// (d = 3, n = 20, m = 20: 24 us as it is, 30 and 26; d = 2, n = 63: 9.7, 12.2 and 10.9).
template <int NMB, int NM0, int NS>
__device__ __forceinline__ void gram_body(const SpecPlan& P, const SpecPtrs& p, int grp, int qb, unsigned char* smem) {
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double2* win = reinterpret_cast<double2*>(smem + window_bytes(P.K1) * wave);
    const bool shift1 = P.d >= 2;
    const int m = P.m, K1 = P.K1, KS = (K1 + 3) >> 2;
    const int R = shift1 ? K1 + 1 : K1, full = R >> 4, rem = R & 15;
    int wa, wb;
    group_range(P, grp, wa, wb);
    const int nw = wb - wa, ng = (rem + 3) >> 2;
    const int q = 16 * qb + col;
    const bool qok = q < m;
    constexpr int CH = NS == 1 ? 8 : 4;      // K steps of V per register set

    double2 acc0[NMB][4], acc1[NS == 2 ? NM0 : 1][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int b = 0; b < NMB; ++b) acc0[b][r] = make_double2(0.0, 0.0);
#pragma unroll
        for (int b = 0; b < (NS == 2 ? NM0 : 1); ++b) acc1[b][r] = make_double2(0.0, 0.0);
    }

    // The group's row blocks in order, shared out over the waves by their products. Up to
    // one full 16-row block per frequency: all full blocks, then all partial ones.
    // More: every full block followed by its part (along h1) of the frequency's partial
    // block, so that a group of one frequency (K1 = 64: four full blocks and one row)
    // splits evenly.
    struct Block {
        int w, r0, s0, s1, ng;
    };
    const int ca = 3 * KS + 12 * NMB, cb = 3 * KS + 3 * ng * NMB;     // MFMAs of a full, a partial block
    int x0, x1;
    if (full > 1) {
        x0 = 2 * (nw * full * wave / kWaves);
        x1 = 2 * (nw * full * (wave + 1) / kWaves);
    } else {
        const int na = full ? nw : 0, nb = rem ? nw : 0;
        auto cut = [&](int k) {
            const int t = (na * ca + nb * cb) * k / kWaves;
            return t < na * ca ? (t + ca / 2) / ca : na + (t - na * ca + cb / 2) / cb;
        };
        x0 = cut(wave);
        x1 = wave + 1 < kWaves ? cut(wave + 1) : na + nb;
    }
    auto block_at = [&](int x) {
        if (full > 1) {
            const int u = x >> 1, w = wa + u / full, v = u % full;
            if (!(x & 1)) return Block{w, 16 * v, 0, KS, 4};
            return Block{w, 16 * full, rem ? KS * v / full : 0, rem ? KS * (v + 1) / full : 0, ng};
        }
        if (full && x < nw) return Block{wa + x, 0, 0, KS, 4};
        return Block{wa + x - (full ? nw : 0), 16 * full, 0, KS, ng};
    };
    // Operands of frequency w are read as buffers of their own K1 m (or NP1) values:
    // rows and samples outside them read as zero, padded columns take kOutside.
    const int row_bytes = 16 * m;
    const int voff = qok ? g * row_bytes + 16 * q : kOutside;
    int uoff[NMB];
#pragma unroll
    for (int b = 0; b < NMB; ++b) {
        const int i = 16 * b + col;   // i >= m: the second m rows, U~[k1 - 1][i - m]
        uoff[b] = i < m ? g * row_bytes + 16 * i
                        : shift1 && i < 2 * m ? (g - 1) * row_bytes + 16 * (i - m) : kOutside;
    }
    auto load_u = [&](double2 (&u)[4], const Block& B, int b) {
        const auto ut = buffer_of(p.ut + (size_t)B.w * K1 * m, K1 * row_bytes);
#pragma unroll
        for (int s = 0; s < 4; ++s) u[s] = buffer_load(ut, uoff[b] + (B.r0 + 4 * s) * row_bytes);
    };

    for (int x = x0; x < x1; ++x) {
        const Block B = block_at(x);
        if (B.s0 == B.s1) continue;
        double2 ua[4], ub[4], ph;
        double yr[4], yi[4];
        toeplitz_rows<CH>(P, p, B.w, B.r0, B.s0, B.s1, voff, false, win, yr, yi, [&] {
            load_u(ua, B, 0);
            ph = p.roots[P.d == 3 ? B.w % P.L : B.w];
        });
        auto gram = [&](const double2 (&uu)[4], auto bc) {
            constexpr int b = decltype(bc)::value;
            acc_t e1 = {0, 0, 0, 0}, e2 = {0, 0, 0, 0}, e3 = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s < B.ng) {
                    e1 = M::fma(uu[s].x, yr[s], e1);
                    e2 = M::fma(uu[s].y, yi[s], e2);
                    e3 = M::fma(uu[s].x - uu[s].y, yr[s] + yi[s], e3);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double gr = e1[r] + e2[r], gi = e3[r] - e1[r] + e2[r];
                double2& a0 = acc0[b][r];
                if constexpr (NS == 1 && b < NM0) {
                    const bool sh = shift1 && 16 * b + M::row(g, r) >= m;
                    const double cr = sh ? 1.0 : ph.x, ci = sh ? 0.0 : ph.y;
                    a0.x = fma(cr, gr, fma(-ci, gi, a0.x));
                    a0.y = fma(cr, gi, fma(ci, gr, a0.y));
                } else {
                    a0.x += gr;
                    a0.y += gi;
                }
                if constexpr (NS == 2 && b < NM0) {
                    double2& a1 = acc1[b][r];
                    a1.x = fma(ph.x, gr, fma(-ph.y, gi, a1.x));
                    a1.y = fma(ph.x, gi, fma(ph.y, gr, a1.y));
                }
            }
        };
        // (the scheduling barriers keep the sums of one block at a time in registers)
        if constexpr (NMB > 1) load_u(ub, B, 1);
        __builtin_amdgcn_sched_barrier(0);
        gram(ua, std::integral_constant<int, 0>{});
        if constexpr (NMB > 2) load_u(ua, B, 2);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NMB > 1) gram(ub, std::integral_constant<int, 1>{});
        if constexpr (NMB > 3) load_u(ub, B, 3);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NMB > 2) gram(ua, std::integral_constant<int, 2>{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NMB > 3) gram(ub, std::integral_constant<int, 3>{});
    }

    // fixed-order sum over the waves and the group's row of partials [i][l][q]
    double2* red = reinterpret_cast<double2*>(smem);   // [wave][block][row][lane]
    double2* out = p.part + (size_t)grp * m * P.ells * m;
    const double2 ph2 = P.d == 3 ? p.roots[wa / P.L] : make_double2(1.0, 0.0);
    auto put = [&](int i, int ell, int qq, double2 v) {
        out[((size_t)i * P.ells + (P.s0 ? ell : ell - 1)) * m + qq] = v;
    };
    auto reduce = [&](const double2 (*acc)[4], auto nbc, bool phased) {
        constexpr int NBK = decltype(nbc)::value, per = NBK * 4 * 64;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NBK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave * per + (b * 4 + r) * 64 + lane] = acc[b][r];
        __syncthreads();
        for (int e = tid; e < per; e += kThreads) {
            const int l = e & 63, br = e >> 6;
            const int i = 16 * (br >> 2) + M::row(l >> 4, br & 3), qq = 16 * qb + (l & 15);
            if (qq >= m || i >= (shift1 ? 2 * m : m)) continue;
            double2 v = red[e];
#pragma unroll
            for (int x = 1; x < kWaves; ++x) {
                v.x += red[x * per + e].x;
                v.y += red[x * per + e].y;
            }
            if (i >= m) {
                if (!phased || NS == 1) put(i - m, 1, qq, v);
            } else if (phased) {
                put(i, P.d, qq, v);          // axis d's phase
            } else {
                if (P.s0) put(i, 0, qq, v);
                if (P.d == 3)
                    put(i, 2, qq, make_double2(fma(ph2.x, v.x, -ph2.y * v.y), fma(ph2.x, v.y, ph2.y * v.x)));
            }
        }
    };
    reduce(acc0, std::integral_constant<int, NMB>{}, NS == 1);
    if constexpr (NS == 2) reduce(acc1, std::integral_constant<int, NM0>{}, true);
}

template <int NMB, int NM0, int NS>
__global__ __launch_bounds__(kThreads, 2) void spectral_gram(SpecPlan P, SpecPtrs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int qb = blockIdx.x % P.nqb, grp = blockIdx.x / P.nqb;
    gram_body<NMB, NM0, NS>(P, p, grp, qb, smem);
}

__device__ __forceinline__ void finish_body(const SpecPlan& P, const SpecPtrs& p, int slice) {
    const int C = P.ells * P.m;
    finish_rows(p.part, P.groups, P.m * C, slice * kFinishOuts, [&](int o, double re, double im) {
        const int i = o / C, c = o - i * C, li = c / P.m, q = c - li * P.m;
        const double s = p.sigma[q];
        p.S[((size_t)li * P.m + i) * P.m + q] = make_double2(re / s, im / s);
    });
}

__global__ __launch_bounds__(kFinishThreads) void spectral_finish(SpecPlan P, SpecPtrs p) {
    finish_body(P, p, blockIdx.x);
}

// ---- products Y = T X, T^* X -------------------------------------------------

// Y~_w[k1][q] = T_w X~_w (or T_w^* X~_w): one 16-row block of one frequency and one
// 16-column block per wave and turn.
__global__ __launch_bounds__(kThreads) void spectral_toeplitz(SpecPlan P, SpecPtrs p, int adjoint) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double2* win = reinterpret_cast<double2*>(smem + window_bytes(P.K1) * wave);
    const int nrb = (P.K1 + 15) >> 4, KS = (P.K1 + 3) >> 2;
    const int units = P.F * P.nqb * nrb;
    for (int u = blockIdx.x * kWaves + wave; u < units; u += gridDim.x * kWaves) {
        const int rb = u % nrb, rest = u / nrb, qb = rest % P.nqb, w = rest / P.nqb;
        const int q = 16 * qb + col;
        double yr[4], yi[4];
        toeplitz_rows<8>(P, p, w, 16 * rb, 0, KS, q < P.m ? 16 * (g * P.m + q) : kOutside, adjoint, win, yr, yi, [] {});
        double2* out = p.ut + (size_t)w * P.K1 * P.m + q;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k1 = 16 * rb + M::row(g, r);
            if (k1 < P.K1 && q < P.m) out[(size_t)k1 * P.m] = make_double2(yr[r], yi[r]);
        }
    }
}

// Inverse transforms: y(k) = sum_w Y~(w) e^{2 pi i w k / L} as A cos + (i B) sin over the
// pairs w < P, A = Y~(w) + Y~(L - w), B = Y~(w) - Y~(L - w). Pair 0 takes A = Y~(0) and, in
// the sine slot with the factors (-1)^k, Y~(P).

// Factors of a lane's output row k at w = 4 s + g.
struct InverseWalk {
    int idx, step, L;
    double alt;
    bool first;       // the next factor is pair 0's
    __device__ __forceinline__ InverseWalk(int k, int g, int L_) {
        L = L_;
        walk_start(k, g, L, idx, step);
        alt = k & 1 ? -1.0 : 1.0;
        first = g == 0;
    }
    __device__ __forceinline__ double2 next(const double2* tab) {
        double2 v = tab[root_slot(idx)];
        idx += step;
        if (idx >= L) idx -= L;
        if (first) v = make_double2(1.0, alt);
        first = false;
        return v;
    }
};

// The two operands of pair w from Y~(w) and its mirror value (one real column, the other
// component in the neighbouring lane).
__device__ __forceinline__ void pair_in(bool zero, bool odd, double a, double b, double& c, double& s) {
    const double x = swap_lane_pair(a - b), y = odd ? x : -x;     // i B
    c = zero ? a : a + b;
    s = zero ? b : y;
}

// Offset of (line t, column q, point j of the transformed axis) in Y (leading dimension
// ld), -1 where there is none.
__device__ __forceinline__ int64_t product_offset(const SpecPlan& P, int64_t ld, int t, int j, int q) {
    const int idx = t * P.P + j;
    return j < P.P && idx < P.N ? idx * ld + q : -1;
}

// One transformed axis (d <= 2): nbc blocks of 8 complex columns c = k1 * m + q of Y~ from
// block nb0. The pairs' operands are staged as [block][w][16 real columns], A then i B.
__global__ __launch_bounds__(kThreads) void spectral_inverse_lines(SpecPlan P, SpecPtrs p, double2* __restrict__ Y,
                                                                   int64_t ld) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int NC = P.K1 * P.m, KS = (P.P + 3) >> 2, J = line_rows(P.P), J4 = 4 * KS;
    const int nblk = (NC + kCols - 1) / kCols, nb0 = blockIdx.x * P.nbi, nbc = min(P.nbi, nblk - nb0);
    double2* tab = reinterpret_cast<double2*>(smem);
    double2* xc = tab + roots_bytes(P.L) / 16;
    double2* xi = xc + (size_t)P.nbi * J * kCols;
    const int tid = threadIdx.x;
    const int tot = nbc * J4 * kCols;
    constexpr int kStage = 4;
    for (int base = 0; base < tot; base += kStage * kThreads) {
        double2 a[kStage], b[kStage];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int e = base + u * kThreads + tid;
            const int cc = e & 7, rest = e >> 3, nb = rest / J4, w = rest - nb * J4, c = kCols * (nb0 + nb) + cc;
            a[u] = b[u] = make_double2(0.0, 0.0);
            if (e < tot && c < NC && w < P.P) {
                a[u] = p.ut[(size_t)w * NC + c];
                b[u] = p.ut[(size_t)(w == 0 ? P.P : P.L - w) * NC + c];
            }
        }
        if (base == 0) fill_roots(tab, P.L);
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int e = base + u * kThreads + tid;
            if (e >= tot) continue;
            const int cc = e & 7, rest = e >> 3, nb = rest / J4, w = rest - nb * J4;
            const int at = (nb * J + w) * kCols + cc;
            const double2 x = a[u], y = b[u];
            xc[at] = w == 0 ? x : make_double2(x.x + y.x, x.y + y.y);
            xi[at] = w == 0 ? y : make_double2(y.y - x.y, x.x - y.x);
        }
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, g = lane >> 4, col = lane & 15;
    const int nrb = (P.P + 15) >> 4;
    for (int it = wave; it < nbc * nrb; it += kWaves) {
        const int nb = it / nrb, rb = it - nb * nrb;
        InverseWalk row(16 * rb + col, g, P.L);
        const double* x1 = reinterpret_cast<const double*>(xc + (size_t)nb * J * kCols) + 16 * g + col;
        const double* x2 = reinterpret_cast<const double*>(xi + (size_t)nb * J * kCols) + 16 * g + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        constexpr int CH = 4;
        double2 a[2][CH];
        double b[2][CH], c[2][CH];
        auto read = [&](int buf, int s) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                b[buf][k] = x1[64 * (s + k)];
                c[buf][k] = x2[64 * (s + k)];
                a[buf][k] = row.next(tab);
            }
        };
        auto mma = [&](int buf, int s) {
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (s + k < KS) {
                    ac = M::fma(a[buf][k].x, b[buf][k], ac);
                    as = M::fma(a[buf][k].y, c[buf][k], as);
                }
        };
        read(0, 0);
        for (int s = 0; s < KS; s += 2 * CH) {
            if (s + CH < KS) read(1, s + CH);
            mma(0, s);
            if (s + 2 * CH < KS) read(0, s + 2 * CH);
            mma(1, s + CH);
        }
        const int cx = kCols * (nb0 + nb) + (col >> 1);
        const int t = cx / P.m, q = cx - t * P.m;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t o = cx < NC ? product_offset(P, ld, t, 16 * rb + M::row(g, r), q) : -1;
            if (o >= 0) reinterpret_cast<double*>(Y)[2 * o + (col & 1)] = ac[r] + as[r];
        }
    }
}

// Two transformed axes (d = 3): the rows k2 of part `split` of one line k1 and nq
// columns: axis 2 into LDS as the operands of axis 3's pairs, then axis 3.
__global__ __launch_bounds__(kThreads) void spectral_inverse_planes(SpecPlan P, SpecPtrs p, double2* __restrict__ Y,
                                                                    int64_t ld) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int per = (P.m + P.nqi - 1) / P.nqi;
    const int split = blockIdx.x % P.isplits, rest0 = blockIdx.x / P.isplits;
    const int q0 = rest0 % per * P.nqi, line = rest0 / per, nq = min(P.nqi, P.m - q0);
    const int k20 = split * P.irows, kn = min(P.irows, P.P - k20);
    const int KS = (P.P + 3) >> 2;
    const size_t rowlen = (size_t)P.K1 * P.m;
    double2* tab = reinterpret_cast<double2*>(smem);
    const int ts = inverse_stride(P.irows, P.nqi);
    double* tc = reinterpret_cast<double*>(tab + roots_bytes(P.L) / 16);      // [w3 pair][k2][q], A
    double* ti = tc + (size_t)4 * KS * ts;                  // i B
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, col = lane & 15;
    const bool odd = lane & 1;
    for (int i = tid; i < (4 * KS - P.P) * ts; i += kThreads) {
        tc[(size_t)P.P * ts + i] = 0.0;
        ti[(size_t)P.P * ts + i] = 0.0;
    }
    // axis 2: columns c = u * nq + q of the pairs u of axis 3, w3 = u and its mirror
    const double* in = reinterpret_cast<const double*>(p.ut);
    const int nc1 = P.P * nq, nb1 = (nc1 + 7) >> 3;
    for (int it = wave; it < nb1 || it == wave; it += kWaves) {      // every wave meets the barrier inside once
        const int c = 8 * it + (col >> 1);
        const bool ok = c < nc1;
        const int u = c / nq, q = c - u * nq;
        const int64_t col0 = 2 * ((int64_t)line * P.m + q0 + q) + (col & 1);
        const int64_t side[2] = {2 * (int64_t)u * (int64_t)rowlen + col0,
                                 2 * (int64_t)(u == 0 ? P.P : P.L - u) * (int64_t)rowlen + col0};
        const int64_t step2 = 2 * (int64_t)P.L * (int64_t)rowlen;      // one frequency of axis 2
        InverseWalk row(k20 + col, g, P.L);
        acc_t ac[2], as[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) ac[i] = as[i] = acc_t{0, 0, 0, 0};
        constexpr int kIn = 3;
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            double a[2][kIn], b[2][kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                const int w = 4 * (s0 + k) + g;
                const bool in_range = ok && w < P.P;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[i][k] = in_range ? in[side[i] + w * step2] : 0.0;
                    b[i][k] = in_range ? in[side[i] + (w == 0 ? P.P : P.L - w) * step2] : 0.0;
                }
            }
            if (it == wave && s0 == 0) {
                fill_roots(tab, P.L);
                __syncthreads();
            }
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                if (s0 + k < KS) {
                    const double2 t = row.next(tab);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        double x, y;
                        pair_in(4 * (s0 + k) + g == 0, odd, a[i][k], b[i][k], x, y);
                        ac[i] = M::fma(t.x, x, ac[i]);
                        as[i] = M::fma(t.y, y, as[i]);
                    }
                }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k2 = M::row(g, r);
            double x, y;
            pair_in(u == 0, odd, ac[0][r] + as[0][r], ac[1][r] + as[1][r], x, y);
            if (ok && k2 < kn) {
                tc[u * ts + 2 * (k2 * nq + q) + (col & 1)] = x;
                ti[u * ts + 2 * (k2 * nq + q) + (col & 1)] = y;
            }
        }
    }
    __syncthreads();
    // axis 3: columns c = k2 * nq + q
    const int nc2 = kn * nq, nb2 = (nc2 + 7) >> 3, nrb = (P.P + 15) >> 4;
    for (int it = wave; it < nb2 * nrb; it += kWaves) {
        const int nb = it / nrb, rb = it - nb * nrb;
        InverseWalk row(16 * rb + col, g, P.L);
        const double* x1 = tc + g * ts + 16 * nb + col;
        const double* x2 = ti + g * ts + 16 * nb + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        for (int s = 0; s < KS; ++s) {
            const double2 t = row.next(tab);
            ac = M::fma(t.x, x1[4 * s * ts], ac);
            as = M::fma(t.y, x2[4 * s * ts], as);
        }
        const int c = 8 * nb + (col >> 1), k2 = c / nq, q = c - k2 * nq;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k3 = 16 * rb + M::row(g, r);
            if (c < nc2 && k3 < P.P)
                reinterpret_cast<double*>(Y)[2 * ((((int64_t)line * P.P + k20 + k2) * P.P + k3) * ld + q0 + q) +
                                             (col & 1)] = ac[r] + as[r];
        }
    }
}

template <typename K>
prony_status_t allow_lds(prony_handle_t h, K kernel, size_t lds) {
    if (lds <= 65536) return PRONY_OK;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    return e == hipSuccess ? PRONY_OK : hip_fail(h, e, "hipFuncSetAttribute");
}

template <int NMB, int NM0, int NS>
prony_status_t launch_gram(prony_handle_t h, const SpecPlan& P, const SpecPtrs& p) {
    const prony_status_t st = allow_lds(h, &spectral_gram<NMB, NM0, NS>, P.lds_gram);
    if (st != PRONY_OK) return st;
    ProfileScope prof(h, "spectral_gram");
    spectral_gram<NMB, NM0, NS><<<P.groups * P.nqb, kThreads, P.lds_gram, h->stream>>>(P, p);
    return PRONY_OK;
}

// (row blocks, those with unshifted rows): m <= 8, 9..16, 17..24, 25..32; d = 1 with
// m > 16 has two unshifted blocks
#define PRONY_GRAM_CASES(X) X(1, 1, 1) X(2, 1, 1) X(2, 2, 1) X(3, 2, 1) X(4, 2, 1) X(1, 1, 2) X(2, 1, 2) X(2, 2, 2) X(3, 2, 2) X(4, 2, 2)

}  // namespace

namespace {

// Two workgroups share a CU's LDS.
size_t lds_budget(prony_handle_t h) { return std::min<size_t>(h->lds_per_block, 80 * 1024); }

// Geometry and forward transforms of a plan with m columns per factor.
bool plan_forward(prony_handle_t h, int d, int n, int m, SpecPlan& P) {
    P = SpecPlan{};
    P.d = d;
    P.n = n;
    P.N = (int)ipow(n + 1, d);
    P.m = m;
    P.pmax = n + 1;
    if (d == 1) {
        // lines of about sqrt(N) points, a multiple of two blocks of pairs
        P.P = 16 * std::max(1, ((int)std::sqrt((double)P.N) + 8) / 16);
        P.K1 = (P.N + P.P - 1) / P.P;
        P.NP1 = 2 * P.K1 - 1;
    } else {
        P.P = n + 1;
        P.K1 = n + 1;
        P.NP1 = 2 * n + 2;
    }
    P.L = 2 * P.P;
    const int64_t F = ipow(P.L, d == 3 ? 2 : 1);
    if (F > (int64_t(1) << 20) || P.K1 > kMaxLines) return false;
    P.F = (int)F;
    P.npb = (P.P + kPairs - 1) / kPairs;
    P.nqb = (m + 15) / 16;
    const size_t budget = lds_budget(h);
    if (d <= 2) {
        // column blocks per workgroup so that its items (a block against two blocks of
        // pairs) share out over the four waves
        const int npi = (P.npb + 1) / 2;
        P.nbw = 1;
        while (P.nbw < 4 && (P.nbw * npi) % kWaves && npi < 4 * kWaves) ++P.nbw;
        auto lds = [&](int nb, int K) { return roots_bytes(P.L) + 16 * kCols * (size_t)nb * line_rows(K); };
        while (P.nbw > 1 && lds(P.nbw, P.P) > budget) --P.nbw;
        P.nbwf = P.nbw;
        while (P.nbwf > 1 && lds(P.nbwf, P.L) > budget) --P.nbwf;
        P.lds_fwd = std::max(lds(P.nbw, P.P), lds(P.nbwf, P.L));
        auto wgs = [&](int64_t cols, int nb) { return (int)(((cols + kCols - 1) / kCols + nb - 1) / nb); };
        P.wgs_x = wgs((int64_t)P.K1 * m, P.nbw);
        P.wgs_f = wgs(P.NP1, P.nbwf);
    } else {
        P.nq = std::min(m, kCols);
        auto lds = [&](int nq, int J, int wp) {
            return roots_bytes(P.L) + 8 * (size_t)((J + 3) & ~3) * plane_stride(wp, nq);
        };
        // one block of pairs per workgroup; fewer pairs where the planes do not fit
        for (P.wp = kPairs; P.wp > 0; P.wp /= 2) {
            P.lds_fwd = std::max(lds(P.nq, P.P, P.wp), lds(1, P.L, P.wp));
            if (P.lds_fwd <= budget) break;
        }
        if (P.wp == 0) return false;
        P.splits = (P.P + P.wp - 1) / P.wp;
        P.wgs_x = P.K1 * ((m + P.nq - 1) / P.nq) * P.splits;
        P.wgs_f = P.NP1 * P.splits;
    }
    return P.lds_fwd <= budget;
}

constexpr size_t kMaxWorkspace = size_t(1) << 30;

}  // namespace

bool spectral_plan(prony_handle_t h, int d, int n, int m, bool s0, SpecPlan& P, bool batched) {
    if (!plan_forward(h, d, n, m, P)) return false;
    P.s0 = s0 ? 1 : 0;
    P.ells = d + P.s0;
    P.nmb = ((d >= 2 ? 2 * m : m) + 15) / 16;
    P.nm0 = P.nqb;
    P.ns = d == 3 || s0 ? 2 : 1;
    const int outer = d == 3 ? P.L : 1;
    // a single instance fills the GPU with two workgroups per CU; a batch member takes
    // workgroups of about 512 products of 16 x 16 x 4 (several microseconds, so that the
    // fixed cost of a workgroup and its row of partials stays small)
    const int R = d >= 2 ? P.K1 + 1 : P.K1, KS = (P.K1 + 3) / 4;
    const int per_w = (R + 15) / 16 * 3 * KS + (R + 3) / 4 * 3 * P.nmb;
    P.gparts = batched ? (int)(((int64_t)P.F / outer * per_w + 511) / 512)
                       : std::max(1, 2 * h->num_cus / (P.nqb * outer));
    P.gparts = std::min(P.F / outer, P.gparts);
    P.groups = outer * P.gparts;
    P.lds_gram = std::max<size_t>(kWaves * window_bytes(P.K1),
                                  (size_t)kWaves * P.nmb * 4 * 64 * sizeof(double2));
    if (P.lds_gram > lds_budget(h)) return false;
    const size_t x = align_up(16 * (size_t)P.F * P.K1 * m, 256);
    P.off_v = x;
    P.off_f = 2 * x;
    P.off_p = P.off_f + align_up(16 * (size_t)P.F * P.NP1, 256);
    P.off_r = P.off_p + align_up(16 * (size_t)P.groups * m * P.ells * m, 256);
    P.ws_bytes = P.off_r + align_up(16 * (size_t)P.L, 256);
    return P.ws_bytes <= kMaxWorkspace;
}

bool spectral_product_plan(prony_handle_t h, int d, int n, int r, SpecPlan& P) {
    if (!plan_forward(h, d, n, r, P)) return false;
    P.pmax = n;
    const size_t budget = lds_budget(h);
    const int KS = (P.P + 3) / 4;
    if (d <= 2) {
        const int nrb = (P.P + 15) / 16;
        auto lds = [&](int nb) { return roots_bytes(P.L) + 2 * 16 * kCols * (size_t)nb * line_rows(P.P); };
        P.nbi = 1;
        while (P.nbi < 4 && (P.nbi * nrb) % kWaves && nrb < 4 * kWaves) ++P.nbi;
        while (P.nbi > 1 && lds(P.nbi) > budget) --P.nbi;
        P.lds_inv = lds(P.nbi);
        P.wgs_i = ((P.K1 * r + kCols - 1) / kCols + P.nbi - 1) / P.nbi;
    } else {
        P.isplits = (P.P + 15) / 16;
        P.irows = (P.P + P.isplits - 1) / P.isplits;
        for (P.nqi = std::min(r, kCols); P.nqi > 0; P.nqi /= 2) {
            P.lds_inv = roots_bytes(P.L) + 2 * 8 * (size_t)(4 * KS) * inverse_stride(P.irows, P.nqi);
            if (P.lds_inv <= budget) break;
        }
        if (P.nqi == 0) return false;
        P.wgs_i = P.K1 * ((r + P.nqi - 1) / P.nqi) * P.isplits;
    }
    if (P.lds_inv > budget) return false;
    const size_t x = align_up(16 * (size_t)P.F * P.K1 * r, 256);
    P.off_v = x;
    P.off_f = 2 * x;
    P.off_r = P.off_f + align_up(16 * (size_t)P.F * P.NP1, 256);
    P.ws_bytes = P.off_r + align_up(16 * (size_t)P.L, 256);
    return P.ws_bytes <= kMaxWorkspace;
}

prony_status_t spectral_product(prony_handle_t h, const SpecPlan& P, unsigned char* ws, const double* f,
                                const double* X, int64_t ldx, bool adjoint, double* Y, int64_t ldy) {
    SpecPtrs p{};
    p.V = reinterpret_cast<const double2*>(X);
    p.v_rs = ldx;
    p.v_cs = 1;
    p.f = reinterpret_cast<const double2*>(f);
    p.ut = reinterpret_cast<double2*>(ws);
    p.vt = reinterpret_cast<double2*>(ws + P.off_v);
    p.ft = reinterpret_cast<double2*>(ws + P.off_f);
    p.roots = reinterpret_cast<double2*>(ws + P.off_r);
    prony_status_t st = allow_lds(h, &spectral_forward_kernel, P.lds_fwd);
    if (st != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_forward");
        spectral_forward_kernel<<<P.wgs_f + P.wgs_x, kThreads, P.lds_fwd, h->stream>>>(P, p, 0);   // the grid and X
    }
    if ((st = check_launch(h, "spectral_forward")) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_toeplitz");
        const int64_t units = (int64_t)P.F * P.nqb * ((P.K1 + 15) / 16);
        const int wgs = (int)std::min<int64_t>((units + kWaves - 1) / kWaves, 4 * (int64_t)h->num_cus);
        spectral_toeplitz<<<wgs, kThreads, kWaves * window_bytes(P.K1), h->stream>>>(P, p, adjoint ? 1 : 0);
    }
    if ((st = check_launch(h, "spectral_toeplitz")) != PRONY_OK) return st;
    if (P.d == 3)
        st = allow_lds(h, &spectral_inverse_planes, P.lds_inv);
    else
        st = allow_lds(h, &spectral_inverse_lines, P.lds_inv);
    if (st != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_inverse");
        double2* y = reinterpret_cast<double2*>(Y);
        if (P.d == 3)
            spectral_inverse_planes<<<P.wgs_i, kThreads, P.lds_inv, h->stream>>>(P, p, y, ldy);
        else
            spectral_inverse_lines<<<P.wgs_i, kThreads, P.lds_inv, h->stream>>>(P, p, y, ldy);
    }
    return check_launch(h, "spectral_inverse");
}

// ---- batches -----------------------------------------------------------------

struct SpecBatch {
    void* ws = nullptr;          // SpecEntry[count], then the instances' workspaces
    int count = 0;
    int fwd_wgs = 0;
    size_t lds_fwd = 0;
    int finish_x = 1;
    struct ClassLaunch {
        int nmb, nm0, ns, first, count, wgs;
        size_t lds;
        double work;             // products of the class
    };
    std::vector<ClassLaunch> launches;
};

namespace {

// One instance of a batch: its plan and operands, its first workgroup in the forward
// launch and in its class's Gram launch.
struct SpecEntry {
    SpecPlan P;
    SpecPtrs p;
    int fwd_begin, gram_begin;
};

// Last entry whose `begin` is at most id.
template <typename Begin>
__device__ __forceinline__ int entry_of(int id, int count, Begin begin) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (begin(mid) <= id)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(kThreads) void spectral_forward_batched(const SpecEntry* __restrict__ entries, int count) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int id = blockIdx.x;
    const SpecEntry& e = entries[entry_of(id, count, [&](int i) { return entries[i].fwd_begin; })];
    forward_body(e.P, e.p, id - e.fwd_begin, smem);
}

template <int NMB, int NM0, int NS>
__global__ __launch_bounds__(kThreads, 2) void spectral_gram_batched(const SpecEntry* __restrict__ entries, int count) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int id = blockIdx.x;
    const SpecEntry& e = entries[entry_of(id, count, [&](int i) { return entries[i].gram_begin; })];
    const int x = id - e.gram_begin;
    gram_body<NMB, NM0, NS>(e.P, e.p, x / e.P.nqb, x % e.P.nqb, smem);
}

__global__ __launch_bounds__(kFinishThreads) void spectral_finish_batched(const SpecEntry* __restrict__ entries) {
    const SpecEntry& e = entries[blockIdx.y];
    if ((int)blockIdx.x * kFinishOuts >= e.P.m * e.P.ells * e.P.m) return;
    finish_body(e.P, e.p, blockIdx.x);
}

template <int NMB, int NM0, int NS>
prony_status_t launch_gram_batched(prony_handle_t h, const SpecEntry* entries, const SpecBatch::ClassLaunch& cl,
                                   hipStream_t stream) {
    const prony_status_t st = allow_lds(h, &spectral_gram_batched<NMB, NM0, NS>, cl.lds);
    if (st != PRONY_OK) return st;
    ProfileScope prof(h, "spectral_gram", stream);
    spectral_gram_batched<NMB, NM0, NS><<<cl.wgs, kThreads, cl.lds, stream>>>(entries + cl.first, cl.count);
    return PRONY_OK;
}

}  // namespace

prony_status_t spectral_batch_free(SpecBatch* b) {
    const prony_status_t st = b->ws && hipFree(b->ws) != hipSuccess ? PRONY_EHIP : PRONY_OK;
    delete b;
    return st;
}

prony_status_t spectral_batch_build(prony_handle_t h, const std::vector<prony_instance_t>& inst, SpecBatch** out) {
    const int count = (int)inst.size();
    std::vector<SpecPlan> plans(count);
    for (int i = 0; i < count; ++i)
        if (!spectral_plan(h, inst[i].d, inst[i].n, inst[i].m, false, plans[i], true))
            return fail(h, PRONY_ENOTSUP, "an instance does not fit the line-spectral form");
    // classes by Gram instantiation; inside a class (and in the forward launch) the
    // largest instances first
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    auto key = [&](int i) { return plans[i].nmb * 16 + plans[i].nm0 * 4 + plans[i].ns; };
    auto work = [&](int i) { return (double)plans[i].F * plans[i].K1 * plans[i].m * (plans[i].K1 + 2 * plans[i].m); };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return key(a) != key(b) ? key(a) > key(b) : work(a) > work(b);
    });
    size_t off = align_up(sizeof(SpecEntry) * (size_t)count, 256);
    std::vector<size_t> base(count);
    for (int pos = 0; pos < count; ++pos) {
        base[pos] = off;
        off += plans[order[pos]].ws_bytes;
    }
    SpecBatch* S = new (std::nothrow) SpecBatch;
    if (!S) return fail(h, PRONY_ENOMEM, "prony_batch_create: out of host memory");
    hipError_t e = hipMalloc(&S->ws, off);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete S;
        return fail(h, PRONY_ENOMEM, std::string("batch workspace allocation failed: ") + hipGetErrorString(e));
    }
    S->count = count;
    std::vector<SpecEntry> host(count);
    int64_t fwd = 0, wgs = 0;
    for (int pos = 0; pos < count; ++pos) {
        const int i = order[pos];
        const SpecPlan& P = plans[i];
        const prony_instance_t& x = inst[i];
        unsigned char* w = static_cast<unsigned char*>(S->ws) + base[pos];
        SpecEntry& E = host[pos];
        E.P = P;
        E.p = SpecPtrs{reinterpret_cast<const double2*>(x.U), reinterpret_cast<const double2*>(x.V), x.m, 1, x.m, 1,
                       reinterpret_cast<const double2*>(x.f), x.sigma, reinterpret_cast<double2*>(w),
                       reinterpret_cast<double2*>(w + P.off_v), reinterpret_cast<double2*>(w + P.off_f),
                       reinterpret_cast<double2*>(w + P.off_p), reinterpret_cast<double2*>(w + P.off_r),
                       reinterpret_cast<double2*>(x.S)};
        E.fwd_begin = (int)fwd;
        fwd += P.wgs_f + 2 * (int64_t)P.wgs_x;
        if (pos == 0 || key(order[pos - 1]) != key(i)) {
            S->launches.push_back({P.nmb, P.nm0, P.ns, pos, 0, 0, 0, 0.0});
            wgs = 0;
        }
        auto& cl = S->launches.back();
        E.gram_begin = (int)wgs;
        wgs += (int64_t)P.groups * P.nqb;
        cl.count += 1;
        cl.wgs = (int)wgs;
        cl.lds = std::max(cl.lds, P.lds_gram);
        cl.work += work(i);
        S->lds_fwd = std::max(S->lds_fwd, P.lds_fwd);
        S->finish_x = std::max(S->finish_x, (P.m * P.ells * P.m + kFinishOuts - 1) / kFinishOuts);
        if (fwd > INT32_MAX || wgs > INT32_MAX) {
            (void)spectral_batch_free(S);
            return fail(h, PRONY_ENOTSUP, "prony_batch_create: too many workgroups");
        }
    }
    S->fwd_wgs = (int)fwd;
    e = hipMemcpyAsync(S->ws, host.data(), sizeof(SpecEntry) * (size_t)count, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        (void)spectral_batch_free(S);
        return hip_fail(h, e, "batch work table upload");
    }
    *out = S;
    return PRONY_OK;
}

prony_status_t spectral_batch_launch(prony_handle_t h, const SpecBatch* S) {
    const SpecEntry* entries = static_cast<const SpecEntry*>(S->ws);
    prony_status_t st = allow_lds(h, &spectral_forward_batched, S->lds_fwd);
    if (st != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_forward");
        spectral_forward_batched<<<S->fwd_wgs, kThreads, S->lds_fwd, h->stream>>>(entries, S->count);
    }
    if ((st = check_launch(h, "spectral_forward_batched")) != PRONY_OK) return st;
    std::vector<double> work;
    for (const auto& cl : S->launches) work.push_back(cl.work);
    st = launch_on_lanes(h, work, [&](int c, hipStream_t stream) {
        const auto& cl = S->launches[c];
        prony_status_t s = PRONY_OK;
        switch (cl.nmb * 16 + cl.nm0 * 4 + cl.ns) {
#define PRONY_CASE(B, B0, K)                                          \
    case B * 16 + B0 * 4 + K:                                         \
        s = launch_gram_batched<B, B0, K>(h, entries, cl, stream);    \
        break;
            PRONY_GRAM_CASES(PRONY_CASE)
#undef PRONY_CASE
            default:
                return fail(h, PRONY_ENOTSUP, "prony_build_S_batched: unexpected spectral plan");
        }
        return s == PRONY_OK ? check_launch(h, "spectral_gram_batched") : s;
    });
    if (st != PRONY_OK) return st;
    {
        ProfileScope prof(h, "pencil_finish");
        spectral_finish_batched<<<dim3(S->finish_x, S->count), kFinishThreads, 0, h->stream>>>(entries);
    }
    return check_launch(h, "spectral_finish_batched");
}

// ---- single instances --------------------------------------------------------

prony_status_t spectral_forward(prony_handle_t h, const SpecPlan& P, const SpecPtrs& ptr, bool factors, bool grid) {
    prony_status_t st = allow_lds(h, &spectral_forward_kernel, P.lds_fwd);
    if (st != PRONY_OK) return st;
    const int first = grid ? 0 : P.wgs_f;
    const int wgs = (grid ? P.wgs_f : 0) + (factors ? 2 * P.wgs_x : 0);
    {
        ProfileScope prof(h, "spectral_forward");
        spectral_forward_kernel<<<wgs, kThreads, P.lds_fwd, h->stream>>>(P, ptr, first);
    }
    return check_launch(h, "spectral_forward");
}

prony_status_t spectral_gram_finish(prony_handle_t h, const SpecPlan& P, const SpecPtrs& ptr) {
    prony_status_t st = PRONY_OK;
    switch (P.nmb * 16 + P.nm0 * 4 + P.ns) {
#define PRONY_CASE(B, B0, S)                   \
    case B * 16 + B0 * 4 + S:                  \
        st = launch_gram<B, B0, S>(h, P, ptr); \
        break;
        PRONY_GRAM_CASES(PRONY_CASE)
#undef PRONY_CASE
        default:
            return fail(h, PRONY_ENOTSUP, "prony_build_S: unexpected spectral plan");
    }
    if (st != PRONY_OK) return st;
    if ((st = check_launch(h, "spectral_gram")) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "pencil_finish");
        const int tot = P.m * P.ells * P.m;
        spectral_finish<<<(tot + kFinishOuts - 1) / kFinishOuts, kFinishThreads, 0, h->stream>>>(P, ptr);
    }
    return check_launch(h, "spectral_finish");
}

}  // namespace prony
