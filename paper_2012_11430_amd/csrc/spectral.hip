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
// of 8 (n+2)^d (n+1)^d m, plus the transforms of U, V and f. Every sum is FP64, but a
// transform's rounding is relative to its whole line (d = 3: plane), so a result's error is
// bounded by the norms of the lines that meet in it, not by its own terms. On samples of even
// size (modes of modulus 1) the errors against extended precision, before (direct sums) and
// here, normwise: S 1.0 to 1.6e-16 and 1.3 to 3.3e-16, products 4.6 to 6.4e-16 and 3.4 to
// 5.5e-16, gradients 1.3 to 2.0e-16 and 2.0 to 4.2e-16; of a gradient's corner points, with
// few terms each, 2e-16 and 1.3 to 3.3e-15 of the value. On damped samples the small entries of
// a product lose digits: d = 2, n = 31, modulus 0.9 per step 5e-16 of the sum of an entry's
// |terms|, 0.8 3e-14 (direct sums 1 to 3e-16).
// d = 1: k = k1 P + k2 is folded into K1 lines of P points, which makes T a two-level
// Toeplitz matrix with f2(p1, p2) = f(p1 P + p2); S_1 is then the phase form along the second
// level.
//
//   spectral_forward  DFTs of U, V and f as real contractions with the cosine and sine
//                     tables on the FP64 matrix cores, folded about the lines' centres:
//                     frequencies w and -w share both sums, points t and -t both factors;
//   spectral_gram     per frequency the Toeplitz product (window of f~_w in LDS) and the
//                     two Gram products, chained in registers: the 16x16 FP64 result
//                     layout (lane group g, element r: row g + 4 r) is the second
//                     operand's layout of K step r, so Y_w never leaves the registers;
//   spectral_finish   fixed-order sum of the groups' partials, Sigma^{-1}.
#include <algorithm>
#include <cmath>
#include <map>
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

// LDS rows of one staged line block (whole groups of K steps) and doubles per row of
// the planes between the two transforms of d = 3 (rows 128 bytes apart modulo 256:
// the rows of two lane groups fall into different banks).
__host__ __device__ inline int line_rows(int K) { return (K + 15) & ~15; }
__host__ __device__ inline int plane_stride(int columns) { return ((2 * columns + 31) & ~31) + 16; }

// Offset in f of the sample (line t, point j of the embedded axis), -1 where there is
// none (the products with T use the samples up to n only). Point j stands for
// p2 = j (j <= P) or j - L.
__device__ __forceinline__ int sample_offset(const SpecPlan& P, int t, int j) {
    const int p1 = t - (P.K1 - 1), p2 = j <= P.P ? j : j - P.L;
    if (P.d == 2) return p1 <= P.pmax && p2 <= P.pmax ? (p1 + P.n) * P.L + p2 + P.n : -1;
    const int p = p1 * P.P + p2;
    return p >= -P.n && p <= P.pmax ? p + P.n : -1;
}

// Folded transforms. A line of P points is transformed about its centre: with
// H = (P + 1) / 2 and t = j + 1/2, point H + j lies at t and point H - 1 - j at -t, so
//     x~(+-w) = C -+ i S,  C = sum_j (x(t) + x(-t)) cos(w t), S = sum_j (x(t) - x(-t)) sin(w t)
// (angles in units of 2 pi / L), half the contraction length of the plain transform. The
// phase of the centre is the same for U and V (and X and Y) and cancels; what is stored
// at L - w is the value at -w. Frequency 0 has no sine row: its slot holds sin(P t) =
// (-1)^j, so that x~(P) = -i S. The sample grid's lines are folded about p = 0: points
// j and -j, j = 0..P, t = j; x~(P) is their sum with the signs (-1)^j. All angles are
// multiples of pi / L.
__host__ __device__ inline int folded_points(int P, bool grid) { return grid ? P + 1 : (P + 1) >> 1; }

// The factors (cos, sin) come from tables in the operand layout of the products, one
// 16-byte load per lane and K step: [16-row block][K step][lane], zero past the contraction's
// end. (Reading them from a table of roots in LDS took 12-15 integer operations per K step,
// more than the products themselves: 300 cycles per step instead of 128.) They depend on P
// only and are kept with the handle. Forward rows are the frequencies w = 16 b + lane % 16,
// the contraction runs over j = 4 s + lane / 16; inverse rows are the points j, the
// contraction runs over the pairs w. Roots: e^{2 pi i j / L}, j < L.
struct TableSizes {
    int ks_f, ks_g, ks_i;              // K steps of the three
    int off_g, off_i, off_r, total;    // in 16-byte entries (factor table first)
};
__host__ __device__ inline TableSizes table_sizes(int P) {
    TableSizes t;
    const int H = folded_points(P, false), blocks = (P + 15) >> 4;
    t.ks_f = (H + 3) >> 2;
    t.ks_g = (P + 4) >> 2;
    t.ks_i = (P + 3) >> 2;
    t.off_g = blocks * t.ks_f * 64;
    t.off_i = t.off_g + ((P + 16) >> 4) * t.ks_g * 64;      // rows 0..P (the adjoint's points)
    t.off_r = t.off_i + ((H + 15) >> 4) * t.ks_i * 64;
    t.total = t.off_r + 2 * P + 8 * 64;      // the K loops load up to 8 steps past a block's end
    return t;
}

__global__ __launch_bounds__(kThreads) void spectral_fill_tables(int P, double2* __restrict__ tab) {
    const TableSizes T = table_sizes(P);
    const int H = folded_points(P, false), L = 2 * P;
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < T.total; i += gridDim.x * kThreads) {
        double2 v = make_double2(0.0, 0.0);
        double s, c;
        if (i >= T.off_r) {
            sincospi(2.0 * (i - T.off_r) / L, &s, &c);
            if (i < T.off_r + L) v = make_double2(c, s);
        } else {
            const int kind = i < T.off_g ? 0 : i < T.off_i ? 1 : 2;
            const int x = i - (kind == 0 ? 0 : kind == 1 ? T.off_g : T.off_i);
            const int ks = kind == 0 ? T.ks_f : kind == 1 ? T.ks_g : T.ks_i;
            const int lane = x & 63, step = (x >> 6) % ks, row = 16 * ((x >> 6) / ks) + (lane & 15);
            const int k = 4 * step + (lane >> 4);
            // angles pi a / L with a = w (2 j + 1), or 2 w j for the grid
            const int w = kind == 2 ? k : row, j = kind == 2 ? row : k;
            const int a = kind == 1 ? 2 * w * j : w * (2 * j + 1);
            sincospi((double)(a % (2 * L)) / L, &s, &c);
            const bool inside = kind == 1 ? w <= P && j <= P : w < P && j < H;
            if (inside) v = make_double2(c, kind != 1 && w == 0 ? (j & 1 ? -1.0 : 1.0) : s);
        }
        tab[i] = v;
    }
}

// x~(w) and x~(-w) (one real column of a complex one, whose other component sits in the
// neighbouring lane) from C and S; w = 0: the frequencies 0 and P (grid: from ny).
__device__ __forceinline__ void pair_out(int w, bool odd, bool grid, double C, double S, double ny, double scale,
                                         double& lo, double& hi) {
    const double x = swap_lane_pair(S), y = odd ? -x : x;
    lo = (w == 0 ? C : C + y) * scale;
    hi = (w == 0 ? (grid ? ny : y) : C - y) * scale;
}

// Sum over the four lane groups of a column's partial sums.
__device__ __forceinline__ double sum_groups(double x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// The transforms are bound by latency at the sizes of one instance (a pass of loads, the
// products of a few items per wave, stores: 9.4 us at d = 2, n = 63, m = 20, 18.4 us at d = 3,
// n = 20, m = 20, of which 10 us are the 50 MB of the counters at the rate of a copy) and by
// memory in a batch (96 instances: 46 us for 199 MB, 40 at that rate). Eight waves per
// workgroup were no faster (19.8 us, batch 68).
//
// Forward transform with one transformed axis (d <= 2): nbc blocks of 8 complex
// columns from block nb0. Columns of a factor: c = line * m + q; of the grid: the
// sample lines t. out[w * NC + c].
template <bool grid>
__device__ __forceinline__ void forward_lines(const SpecPlan& P, const double2* __restrict__ src, int64_t rs,
                                              int64_t cs, double2* __restrict__ out,
                                              const double2* __restrict__ tables, int nb0, int nbc,
                                              unsigned char* smem) {
    const int mc = grid ? 1 : P.m;
    const int NC = grid ? P.NP1 : P.K1 * P.m;
    const int K = folded_points(P.P, grid), KS = (K + 3) >> 2, J = line_rows(K);
    double2* xs = reinterpret_cast<double2*>(smem);     // sums, [block][j][8 columns]
    double2* xd = xs + (size_t)nbc * J * kCols;         // differences
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // an item is a 16-row block of frequency pairs against up to two column blocks; the
    // first item's factors are requested before the inputs
    constexpr int NB = 2, CH = 8;
    const int items = P.npb * ((nbc + NB - 1) / NB);
    const double2* tab = tables + (grid ? table_sizes(P.P).off_g : 0) + lane;
    double2 tn[CH];
    auto load_t = [&](int it, int s) {
        const double2* x = tab + (size_t)(it % P.npb * KS + s) * 64;
#pragma unroll
        for (int k = 0; k < CH; ++k) tn[k] = x[64 * k];
    };
    load_t(wave, 0);
    // the inputs in tiles of 16 points x 8 columns per half workgroup, lanes along the
    // axis that is contiguous in memory, 8 loads in flight
    const bool jfast = grid || rs < cs;
    const int e = tid & 127, jl = jfast ? e & 15 : e >> 3, cc = jfast ? e >> 4 : e & 7;
    const int half = tid >> 7, per = (J / 16 + 1) / 2, turns = nbc * per;   // turns of both halves
    constexpr int kStage = 4;
    for (int base = 0; base < turns; base += kStage) {
        double2 a[kStage], b[kStage];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            a[u] = b[u] = make_double2(0.0, 0.0);
            if (base + u < turns) {
                const int nb = (base + u) / per, j = 16 * (2 * (base + u - nb * per) + half) + jl;
                const int c = kCols * (nb0 + nb) + cc;
                if (c < NC && j < K) {
                    if (grid) {
                        const int oa = sample_offset(P, c, j);
                        const int ob = j > 0 && j < P.P ? sample_offset(P, c, P.L - j) : -1;
                        if (oa >= 0) a[u] = src[oa];
                        if (ob >= 0) b[u] = src[ob];
                    } else {
                        const int line = c / mc, q = c - line * mc;
                        const int ia = line * P.P + K + j, ib = line * P.P + K - 1 - j;
                        if (K + j < P.P && ia < P.N) a[u] = src[ia * rs + q * cs];
                        if (ib < P.N) b[u] = src[ib * rs + q * cs];
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kStage; ++u)
            if (base + u < turns) {
                const int nb = (base + u) / per, j = 16 * (2 * (base + u - nb * per) + half) + jl;
                if (j < J) {
                    xs[(nb * J + j) * kCols + cc] = make_double2(a[u].x + b[u].x, a[u].y + b[u].y);
                    xd[(nb * J + j) * kCols + cc] = make_double2(a[u].x - b[u].x, a[u].y - b[u].y);
                }
            }
    }
    __syncthreads();
    const bool odd = lane & 1;
    const double scale = grid ? 1.0 / P.F : 1.0, alt = g & 1 ? -1.0 : 1.0;
    for (int it = wave; it < items; it += kWaves) {
        const int pb = it % P.npb, nbf = it / P.npb * NB, cnt = min(NB, nbc - nbf);
        const double* x1 = reinterpret_cast<const double*>(xs + (size_t)nbf * J * kCols) + 16 * g + col;
        const double* x2 = reinterpret_cast<const double*>(xd + (size_t)nbf * J * kCols) + 16 * g + col;
        acc_t ac[NB], as[NB];
        double ny[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            ac[i] = as[i] = acc_t{0, 0, 0, 0};
            ny[i] = 0.0;
        }
        for (int s = 0; s < KS; s += CH) {
            double2 t[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) t[k] = tn[k];
            if (s + CH < KS)
                load_t(it, s + CH);
            else if (it + kWaves < items)
                load_t(it + kWaves, 0);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (i >= cnt) break;
                const double* y1 = x1 + 16 * J * i + 64 * s;
                const double* y2 = x2 + 16 * J * i + 64 * s;
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    if (s + k >= KS) break;
                    const double b = y1[64 * k];
                    ac[i] = M::fma(t[k].x, b, ac[i]);
                    as[i] = M::fma(t[k].y, y2[64 * k], as[i]);
                    if (grid) ny[i] = fma(alt, b, ny[i]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (i >= cnt) break;
            if (grid) ny[i] = sum_groups(ny[i]);
            const int c = kCols * (nb0 + nbf + i) + (col >> 1);
            double* o = reinterpret_cast<double*>(out) + 2 * c + (col & 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int w = 16 * pb + M::row(g, r);
                double lo, hi;
                pair_out(w, odd, grid, ac[i][r], as[i][r], ny[i], scale, lo, hi);
                if (w < P.P && c < NC) {
                    o[(size_t)w * NC * 2] = lo;
                    o[(size_t)(w == 0 ? P.P : P.L - w) * NC * 2] = hi;
                }
            }
        }
    }
}

// Forward transform with two transformed axes (d = 3): the plane (axes 2, 3) of line
// `line` and nq complex columns from column q0: axis 3 at the pairs split * wp ..
// (and their mirrors) into LDS, then axis 2. out[(w2 L + w3) * rowlen + line * mc + q].
template <bool grid>
__device__ __forceinline__ void forward_planes(const SpecPlan& P, const double2* __restrict__ src, int64_t rs,
                                               int64_t cs, double2* __restrict__ out,
                                               const double2* __restrict__ tables, int line, int q0, int nq,
                                               int split, unsigned char* smem) {
    const int mc = grid ? 1 : P.m;
    const size_t rowlen = grid ? P.NP1 : (size_t)P.K1 * P.m;
    const int J = grid ? P.L : P.P;                     // points of an axis
    const int K = folded_points(P.P, grid), KS = (K + 3) >> 2;
    const int w0 = split * 16, wn = min(16, P.P - w0);
    double* t1 = reinterpret_cast<double*>(smem);       // [j2][2 u + side][q] complex
    const int ts = plane_stride(2 * wn * nq);
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool odd = lane & 1;
    const double alt = g & 1 ? -1.0 : 1.0;
    const double2* tab = tables + (grid ? table_sizes(P.P).off_g : 0) + lane;
    const double* in = reinterpret_cast<const double*>(src);
    const int jskip = P.pmax == P.n ? P.P : -1;      // the point p = n + 1 of an axis
    // row J is zero: the second operand of points without a mirror
    for (int i = tid; i < ts; i += kThreads) t1[(size_t)J * ts + i] = 0.0;

    // axis 3: columns c = j2 * nq + q in blocks of 8, NBI blocks per pass, kIn K steps of
    // factors and inputs at a time; the next ones are requested before the products
    constexpr int NBI = grid ? 1 : 2, kIn = grid ? 6 : 3;
    const int nc1 = J * nq, nb1 = (nc1 + 7) >> 3, items1 = (nb1 + NBI - 1) / NBI;
    const float rnq = 1.0f / nq;
    auto div_nq = [&](int c) { return (int)((c + 0.5f) * rnq); };     // c < 2^14: exact
    struct Item {
        bool live[NBI];          // columns of the plane
        int o1[NBI];             // their places in an LDS row
        const double* x[NBI];    // their inputs, null where there are none
    };
    auto item_at = [&](int it, Item& I) {
#pragma unroll
        for (int i = 0; i < NBI; ++i) {
            const int c = 8 * (it * NBI + i) + (col >> 1);
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
    // inputs of K steps s0 .. : offsets of the points t and -t from a column's first input
    const int64_t up = grid ? 2 : 2 * rs;
    const int64_t oa0 = (grid ? g : K + g) * up, ob0 = (grid ? -g : K - 1 - g) * up;
    auto load = [&](double (&a)[NBI][kIn], double (&b)[NBI][kIn], const Item& I, int s0) {
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const int j = 4 * (s0 + k) + g;
            const bool ka = grid ? j < K && j != jskip : j < K && K + j < P.P, kb = grid ? j > 0 && j < P.P : j < K;
            const int64_t d = 4 * (s0 + k) * up;
#pragma unroll
            for (int i = 0; i < NBI; ++i) {
                a[i][k] = I.x[i] && ka ? I.x[i][oa0 + d] : 0.0;
                b[i][k] = I.x[i] && kb ? I.x[i][ob0 - d] : 0.0;
            }
        }
    };
    double2 t[kIn];
    auto load_t = [&](int pb, int s0) {
        const double2* x = tab + (size_t)(pb * KS + s0) * 64;
#pragma unroll
        for (int k = 0; k < kIn; ++k) t[k] = x[64 * k];
    };
    Item item;
    double a[NBI][kIn], b[NBI][kIn];
    load_t(split, 0);
    item_at(wave, item);
    load(a, b, item, 0);
    for (int it = wave; it < items1; it += kWaves) {
        acc_t ac[NBI], as[NBI];
        double ny[NBI];
#pragma unroll
        for (int i = 0; i < NBI; ++i) {
            ac[i] = as[i] = acc_t{0, 0, 0, 0};
            ny[i] = 0.0;
        }
        Item next;
        item_at(it + kWaves, next);
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            double an[NBI][kIn], bn[NBI][kIn];
            if (KS > kIn) load_t(split, s0);
            // the next K steps or the next item's first ones
            const bool more = s0 + kIn < KS;
            load(an, bn, more ? item : next, more ? s0 + kIn : 0);
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                if (s0 + k < KS)
#pragma unroll
                    for (int i = 0; i < NBI; ++i) {
                        const double s = a[i][k] + b[i][k];
                        ac[i] = M::fma(t[k].x, s, ac[i]);
                        as[i] = M::fma(t[k].y, a[i][k] - b[i][k], as[i]);
                        if (grid) ny[i] = fma(alt, s, ny[i]);
                    }
#pragma unroll
            for (int i = 0; i < NBI; ++i)
#pragma unroll
                for (int k = 0; k < kIn; ++k) {
                    a[i][k] = an[i][k];
                    b[i][k] = bn[i][k];
                }
        }
#pragma unroll
        for (int i = 0; i < NBI; ++i) {
            if (grid) ny[i] = sum_groups(ny[i]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int u = M::row(g, r);
                double lo, hi;
                pair_out(w0 + u, odd, grid, ac[i][r], as[i][r], ny[i], 1.0, lo, hi);
                if (item.live[i] && u < wn) {
                    t1[item.o1[i] + 4 * u * nq] = lo;
                    t1[item.o1[i] + (4 * u + 2) * nq] = hi;
                }
            }
        }
        item = next;
    }

    // axis 2: columns c = (2 u + side) * nq + q of the LDS rows j2; an item is a 16-row
    // block of pairs against NB2 column blocks. Per item and kIn K steps the factors and
    // the rows of t and -t (row J, zero, where there is none)
    constexpr int NB2 = grid ? 1 : 2;
    const int nc2 = 2 * wn * nq, nb2 = (nc2 + 7) >> 3, ng2 = (nb2 + NB2 - 1) / NB2, items2 = ng2 * P.npb;
    const double scale = grid ? 1.0 / P.F : 1.0;
    const int64_t step2 = 2 * (int64_t)P.L * rowlen;          // one frequency of axis 2
    // the items of a block of pairs go to the waves in turn, block after block
    if (wave < items2) load_t(wave / ng2, 0);
    __syncthreads();
    int ra[kIn], rb[kIn];
    auto rows_at = [&](int s0) {
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const int j = 4 * (s0 + k) + g;
            ra[k] = ((grid ? j < K : j < K && K + j < J) ? (grid ? j : K + j) : J) * ts + col;
            rb[k] = ((grid ? j > 0 && j < P.P : j < K) ? (grid ? J - j : K - 1 - j) : J) * ts + col;
        }
    };
    rows_at(0);
    int pb_held = wave / ng2;        // the block whose factors t holds
    for (int it = wave; it < items2; it += kWaves) {
        const int pb = it / ng2, ng = it - pb * ng2;
        acc_t ac[NB2], as[NB2];
        double ny[NB2];
        int at[NB2];
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
            ac[i] = as[i] = acc_t{0, 0, 0, 0};
            ny[i] = 0.0;
            // columns past the last read the last block again and are not stored
            at[i] = 16 * min(ng * NB2 + i, nb2 - 1);
        }
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            if (KS > kIn || pb != pb_held) load_t(pb, s0);
            if (KS > kIn) rows_at(s0);
            double p[kIn][NB2], q[kIn][NB2];
#pragma unroll
            for (int k = 0; k < kIn; ++k)
#pragma unroll
                for (int i = 0; i < NB2; ++i) {
                    p[k][i] = t1[ra[k] + at[i]];
                    q[k][i] = t1[rb[k] + at[i]];
                }
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                if (s0 + k < KS)
#pragma unroll
                    for (int i = 0; i < NB2; ++i) {
                        const double c = p[k][i] + q[k][i];
                        ac[i] = M::fma(t[k].x, c, ac[i]);
                        as[i] = M::fma(t[k].y, p[k][i] - q[k][i], as[i]);
                        if (grid) ny[i] = fma(alt, c, ny[i]);
                    }
        }
        pb_held = pb;
        // the next item's factors, should it start another block
        if (KS <= kIn && it + kWaves < items2 && (it + kWaves) / ng2 != pb) {
            pb_held = (it + kWaves) / ng2;
            load_t(pb_held, 0);
        }
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
            if (grid) ny[i] = sum_groups(ny[i]);
            const int c = 8 * (ng * NB2 + i) + (col >> 1);
            const int wl = div_nq(c), qq = c - wl * nq, w3p = w0 + (wl >> 1);
            const int w3 = wl & 1 ? (w3p == 0 ? P.P : P.L - w3p) : w3p;
            // rows w2 = 16 pb + g + 4 r and their mirrors
            double* o = reinterpret_cast<double*>(out) + 2 * ((size_t)w3 * rowlen + (size_t)line * mc + q0 + qq) + (col & 1);
            const int wg = 16 * pb + g;
            double* olo = o + wg * step2;
            double* ohi = o + (P.L - wg) * step2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int w2 = wg + 4 * r;
                double lo, hi;
                pair_out(w2, odd, grid, ac[i][r], as[i][r], ny[i], scale, lo, hi);
                if (w2 < P.P && c < nc2) {
                    olo[4 * r * step2] = lo;
                    (w2 == 0 ? o + P.P * step2 : ohi - 4 * r * step2)[0] = hi;
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
    const int x = grid ? id : id - P.wgs_f - (second ? P.wgs_x : 0);
    const double2* src = grid ? p.f : second ? p.U : p.V;
    const int64_t rs = second ? p.u_rs : p.v_rs, cs = second ? p.u_cs : p.v_cs;
    double2* out = grid ? p.ft : second ? p.ut : p.vt;
    if (P.d == 3) {
        const int split = x % P.splits, rest = x / P.splits;
        if (grid) {
            forward_planes<true>(P, src, 0, 0, out, p.tab, rest, 0, 1, split, smem);
        } else {
            const int per = (P.m + P.nq - 1) / P.nq;   // column blocks of a line
            const int qb = rest % per, line = rest / per;
            forward_planes<false>(P, src, rs, cs, out, p.tab, line, qb * P.nq, min(P.nq, P.m - qb * P.nq), split, smem);
        }
    } else if (grid) {
        const int nblk = (P.NP1 + kCols - 1) / kCols;
        forward_lines<true>(P, src, 0, 0, out, p.tab, x * P.nbwf, min(P.nbwf, nblk - x * P.nbwf), smem);
    } else {
        const int nblk = (P.K1 * P.m + kCols - 1) / kCols;
        forward_lines<false>(P, src, rs, cs, out, p.tab, x * P.nbw, min(P.nbw, nblk - x * P.nbw), smem);
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
// one's loads overlap the other's products.
//   d = 3, n = 20, m = 20 takes 21.7 us (tiles of the row-extended product: 270), the matrix
// cores busy 45 % of it; the rest is the latency of a block's loads, f~ through LDS, with two
// waves per SIMD, and eight vector instructions per product. d = 2, n = 63: 10.8 us (tiles:
// 65; one wave per SIMD, matrix cores 30 %). Not faster: requesting the next row block's operands before the Gram products, or the
// full and partial block of a frequency together on shared V operands (registers spill:
// 30 and 26 against 24 us at the time); blocks dealt to the waves in turn (24.4 against 21.7
// us) or to the wave with the least (25.7), so the longest wave is not the bound.
template <int NMB, int NM0, int NS>
__device__ __forceinline__ void gram_body(const SpecPlan& P, const SpecPtrs& p, int grp, int qb, unsigned char* smem) {
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double2* win = reinterpret_cast<double2*>(smem + window_bytes(P.K1) * wave);
    const double2* roots = p.tab + table_sizes(P.P).off_r;
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
            ph = roots[P.d == 3 ? B.w % P.L : B.w];
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
    const double2 ph2 = P.d == 3 ? roots[wa / P.L] : make_double2(1.0, 0.0);
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

// Three launches per product, each bound by latency: d = 2, n = 63, r = 40 9.4 + 9 + 6 us
// (tiles of the whole product: 85), d = 3, n = 20, r = 1 10 + 7.5 + 7 us (vector kernel: 47).
// One column takes the same 16-column blocks: the matrix work is not what it waits for.
//
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

// A transform spreads a NaN, an infinity or a sum past the largest double over all the points
// of its lines. Where a result is not finite it is therefore formed again from the inputs, so
// that it depends on its own terms only; a sum that is NaN ends there. The offset of index
// (k1, k2, k3) in the sample grid, from that of the index 0 in every axis:
__device__ __forceinline__ bool is_finite(double x) { return fabs(x) <= 1.7976931348623157e308; }
__device__ __forceinline__ int64_t grid_offset(const SpecPlan& P, int k) {
    const int E = P.n + 1, Q = 2 * P.n + 2;
    if (P.d == 1) return k;
    if (P.d == 2) return (int64_t)(k / E) * Q + k % E;
    return ((int64_t)(k / (E * E)) * Q + k / E % E) * Q + k % E;
}
__device__ __forceinline__ int64_t grid_centre(const SpecPlan& P) {
    const int64_t Q = 2 * P.n + 2;
    return P.n * (P.d == 1 ? 1 : P.d == 2 ? 1 + Q : 1 + Q + Q * Q);
}

// Whether any thread's `bad` is set (`flag`, in LDS, is zero before); if so, what the
// workgroup stored before is visible to all of it. Else no wait for the stores: a barrier that
// waits for them, like __syncthreads_or, took 1 us of a gradient's 16 to 35.
__device__ __forceinline__ bool any_bad(bool bad, int* flag) {
    if (bad) *flag = 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (!*static_cast<volatile int*>(flag)) return false;
    __threadfence_block();
    __syncthreads();
    return true;
}

// The components of (T X)[k, q] or (T^* X)[k, q] at `y` that are not finite, from the
// inputs: N terms, loads in flight for several at a time.
__device__ __forceinline__ void direct_product(const SpecPlan& P, const SpecPtrs& p, bool adjoint, int k, int q,
                                               double2* y) {
    const bool fix_x = !is_finite(y->x), fix_y = !is_finite(y->y);
    if (!fix_x && !fix_y) return;
    const int64_t row = grid_centre(P) + (adjoint ? -grid_offset(P, k) : grid_offset(P, k));
    const double2* x = p.V + q * p.v_cs;
    const int line = P.d == 1 ? P.N : P.n + 1, step = adjoint ? 1 : -1;
    double re = 0.0, im = 0.0;
    for (int h0 = 0; h0 < P.N; h0 += line) {
        const double2* f = p.f + row + step * grid_offset(P, h0);
        const double2* xl = x + h0 * p.v_rs;
#pragma unroll 8
        for (int h = 0; h < line; ++h) {
            const double2 a = f[(int64_t)step * h], b = xl[h * p.v_rs];
            const double ay = adjoint ? -a.y : a.y;
            re = fma(a.x, b.x, fma(-ay, b.y, re));
            im = fma(a.x, b.y, fma(ay, b.x, im));
        }
        if ((!fix_x || re != re) && (!fix_y || im != im)) break;
    }
    if (fix_x) y->x = re;
    if (fix_y) y->y = im;
}

// Inverse transforms about the line's centre (see the folded forward ones): at t = j + 1/2
//     y(+-t) = C +- S,  C = sum_w A cos(w t), S = sum_w (i B) sin(w t)
// over the pairs w < P, A = Y~(w) + Y~(-w), B = Y~(w) - Y~(-w). Pair 0: A = Y~(0), and in the
// sine slot, with sin(P t) = (-1)^j, B = Y~(P).

// The two operands A and i B of pair w from Y~(w) and Y~(-w) (one real column, the other
// component in the neighbouring lane).
__device__ __forceinline__ void pair_in(bool zero, bool odd, double a, double b, double& c, double& s) {
    const double x = swap_lane_pair(zero ? b : a - b);
    c = zero ? a : a + b;
    s = odd ? x : -x;
}

// One transformed axis (d <= 2): nbc blocks of 8 complex columns c = k1 * m + q of Y~ from
// block nb0. The pairs' operands are staged as [block][w][16 real columns], A then i B.
__global__ __launch_bounds__(kThreads) void spectral_inverse_lines(SpecPlan P, SpecPtrs p, double2* __restrict__ Y,
                                                                   int64_t ld, int adjoint) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int bad_flag;
    if (threadIdx.x == 0) bad_flag = 0;
    const int NC = P.K1 * P.m, KS = (P.P + 3) >> 2, J = line_rows(P.P), H = folded_points(P.P, false);
    const int nblk = (NC + kCols - 1) / kCols, nb0 = blockIdx.x * P.nbi, nbc = min(P.nbi, nblk - nb0);
    double2* xc = reinterpret_cast<double2*>(smem);
    double2* xi = xc + (size_t)P.nbi * J * kCols;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nrb = (H + 15) >> 4;
    // the first item's factors are requested before the inputs
    constexpr int CH = 8;
    const double2* tab = p.tab + table_sizes(P.P).off_i + lane;
    double2 fn[CH];
    auto load_t = [&](int it, int s) {
        const double2* x = tab + (size_t)(it % nrb * KS + s) * 64;
#pragma unroll
        for (int k = 0; k < CH; ++k) fn[k] = x[64 * k];
    };
    load_t(wave, 0);
    // lane (w, column) of tiles of 32 pairs x 8 columns
    const int cc = tid & 7, wl = tid >> 3, per = (J + 31) / 32, turns = nbc * per;
    constexpr int kStage = 4;
    for (int base = 0; base < turns; base += kStage) {
        double2 a[kStage], b[kStage];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int nb = (base + u) / per, w = 32 * (base + u - nb * per) + wl, c = kCols * (nb0 + nb) + cc;
            a[u] = b[u] = make_double2(0.0, 0.0);
            if (base + u < turns && c < NC && w < P.P) {
                a[u] = p.ut[(size_t)w * NC + c];
                b[u] = p.ut[(size_t)(w == 0 ? P.P : P.L - w) * NC + c];
            }
        }
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int nb = (base + u) / per, w = 32 * (base + u - nb * per) + wl;
            if (base + u >= turns || w >= J) continue;
            const int at = (nb * J + w) * kCols + cc;
            const double2 x = a[u], y = b[u];
            const double2 d = w == 0 ? y : make_double2(x.x - y.x, x.y - y.y);
            xc[at] = w == 0 ? x : make_double2(x.x + y.x, x.y + y.y);
            xi[at] = make_double2(-d.y, d.x);
        }
    }
    __syncthreads();
    bool bad = false;
    for (int it = wave; it < nbc * nrb; it += kWaves) {
        const int nb = it / nrb, rb = it - nb * nrb;
        const double* x1 = reinterpret_cast<const double*>(xc + (size_t)nb * J * kCols) + 16 * g + col;
        const double* x2 = reinterpret_cast<const double*>(xi + (size_t)nb * J * kCols) + 16 * g + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        for (int s = 0; s < KS; s += CH) {
            double2 f[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) f[k] = fn[k];
            if (s + CH < KS)
                load_t(it, s + CH);
            else if (it + kWaves < nbc * nrb)
                load_t(it + kWaves, 0);
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                if (s + k >= KS) break;
                ac = M::fma(f[k].x, x1[64 * (s + k)], ac);
                as = M::fma(f[k].y, x2[64 * (s + k)], as);
            }
        }
        const int cx = kCols * (nb0 + nb) + (col >> 1);
        const int t = cx / P.m, q = cx - t * P.m;
        double* o = reinterpret_cast<double*>(Y) + 2 * q + (col & 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 16 * rb + M::row(g, r);
            const int ia = t * P.P + H + j, ib = t * P.P + H - 1 - j;
            if (cx < NC && j < H) {
                const double ya = ac[r] + as[r], yb = ac[r] - as[r];
                bad = bad || !is_finite(ya) || !is_finite(yb);
                if (H + j < P.P && ia < P.N) o[2 * ia * ld] = ya;
                if (ib < P.N) o[2 * ib * ld] = yb;
            }
        }
    }
    // the workgroup's results that are not finite, a thread each
    if (__builtin_expect(any_bad(bad, &bad_flag), 0))
        for (int e = tid; e < kCols * nbc * P.P; e += kThreads) {
            const int c = kCols * nb0 + e / P.P, t = c / P.m, q = c - t * P.m, i = t * P.P + e % P.P;
            if (c < NC && i < P.N) direct_product(P, p, adjoint, i, q, Y + i * ld + q);
        }
}

// Two transformed axes (d = 3): the rows k2 = H + j, H - 1 - j, j in part `split`, of one
// line k1 and nq columns: axis 2 into LDS as the operands of axis 3's pairs, then axis 3.
__global__ __launch_bounds__(kThreads) void spectral_inverse_planes(SpecPlan P, SpecPtrs p, double2* __restrict__ Y,
                                                                    int64_t ld, int adjoint) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int bad_flag;
    if (threadIdx.x == 0) bad_flag = 0;
    const int per = (P.m + P.nqi - 1) / P.nqi;
    const int split = blockIdx.x % P.isplits, rest0 = blockIdx.x / P.isplits;
    const int q0 = rest0 % per * P.nqi, line = rest0 / per, nq = min(P.nqi, P.m - q0);
    const int H = folded_points(P.P, false), j0 = split * P.irows, kn = min(P.irows, H - j0);
    const int KS = (P.P + 3) >> 2;
    const size_t rowlen = (size_t)P.K1 * P.m;
    const int ts = plane_stride(2 * P.irows * P.nqi);
    double* tc = reinterpret_cast<double*>(smem);       // [w3 pair][2 j + side][q], A
    double* ti = tc + (size_t)4 * KS * ts;              // i B
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool odd = lane & 1;
    const double2* tab = p.tab + table_sizes(P.P).off_i;
    // factors of the part's rows j0 + col (they need not start a block of the table)
    const int jr = min(j0 + col, H - 1);
    const double2* tab2 = tab + (size_t)(jr >> 4) * KS * 64 + 16 * g + (jr & 15);
    for (int i = tid; i < (4 * KS - P.P) * ts; i += kThreads) {
        tc[(size_t)P.P * ts + i] = 0.0;
        ti[(size_t)P.P * ts + i] = 0.0;
    }
    // axis 2: columns c = u * nq + q of the pairs u of axis 3, w3 = u and its mirror
    const double* in = reinterpret_cast<const double*>(p.ut);
    const int nc1 = P.P * nq, nb1 = (nc1 + 7) >> 3;
    for (int it = wave; it < nb1; it += kWaves) {
        const int c = 8 * it + (col >> 1);
        const bool ok = c < nc1;
        const int u = c / nq, q = c - u * nq;
        const int64_t col0 = 2 * ((int64_t)line * P.m + q0 + q) + (col & 1);
        const int64_t side[2] = {2 * (int64_t)u * (int64_t)rowlen + col0,
                                 2 * (int64_t)(u == 0 ? P.P : P.L - u) * (int64_t)rowlen + col0};
        const int64_t step2 = 2 * (int64_t)P.L * (int64_t)rowlen;      // one frequency of axis 2
        acc_t ac[2], as[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) ac[i] = as[i] = acc_t{0, 0, 0, 0};
        constexpr int kIn = 3;
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            double a[2][kIn], b[2][kIn];
            double2 t[kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                t[k] = tab2[64 * (s0 + k)];
                const int w = 4 * (s0 + k) + g;
                const bool in_range = ok && w < P.P;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[i][k] = in_range ? in[side[i] + w * step2] : 0.0;
                    b[i][k] = in_range ? in[side[i] + (w == 0 ? P.P : P.L - w) * step2] : 0.0;
                }
            }
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                if (s0 + k < KS) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        double x, y;
                        pair_in(4 * (s0 + k) + g == 0, odd, a[i][k], b[i][k], x, y);
                        ac[i] = M::fma(t[k].x, x, ac[i]);
                        as[i] = M::fma(t[k].y, y, as[i]);
                    }
                }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = M::row(g, r);
            double x[2], y[2];       // rows H + j0 + j and H - 1 - j0 - j
            pair_in(u == 0, odd, ac[0][r] + as[0][r], ac[1][r] + as[1][r], x[0], y[0]);
            pair_in(u == 0, odd, ac[0][r] - as[0][r], ac[1][r] - as[1][r], x[1], y[1]);
            if (ok && j < kn)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int at = u * ts + 2 * ((2 * j + h) * nq + q) + (col & 1);
                    tc[at] = x[h];
                    ti[at] = y[h];
                }
        }
    }
    __syncthreads();
    // axis 3: columns c = (2 j + side) * nq + q
    const int nc2 = 2 * kn * nq, nb2 = (nc2 + 7) >> 3, nrb = (H + 15) >> 4;
    bool bad = false;
    for (int it = wave; it < nb2 * nrb; it += kWaves) {
        const int nb = it / nrb, rb = it - nb * nrb;
        const double2* tab3 = tab + (size_t)rb * KS * 64 + lane;
        const double* x1 = tc + g * ts + 16 * nb + col;
        const double* x2 = ti + g * ts + 16 * nb + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        constexpr int CH = 3;
        for (int s = 0; s < KS; s += CH) {
            double2 t[CH];
            double b[CH], c[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int row_s = 4 * min(s + k, KS - 1) * ts;
                b[k] = x1[row_s];
                c[k] = x2[row_s];
                t[k] = tab3[64 * (s + k)];
            }
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (s + k < KS) {
                    ac = M::fma(t[k].x, b[k], ac);
                    as = M::fma(t[k].y, c[k], as);
                }
        }
        const int c = 8 * nb + (col >> 1), kk = c / nq, q = c - kk * nq;
        const int k2 = kk & 1 ? H - 1 - j0 - (kk >> 1) : H + j0 + (kk >> 1);
        double* o = reinterpret_cast<double*>(Y) + 2 * (((int64_t)line * P.P + k2) * P.P * ld + q0 + q) + (col & 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 16 * rb + M::row(g, r);
            if (c < nc2 && k2 < P.P && j < H) {
                const double ya = ac[r] + as[r], yb = ac[r] - as[r];
                bad = bad || !is_finite(ya) || !is_finite(yb);
                if (H + j < P.P) o[2 * (H + j) * ld] = ya;
                o[2 * (H - 1 - j) * ld] = yb;
            }
        }
    }
    if (__builtin_expect(any_bad(bad, &bad_flag), 0))
        for (int e = tid; e < nc2 * P.P; e += kThreads) {
            const int c = e / P.P, k3 = e % P.P, kk = c / nq, q = q0 + c - kk * nq;
            const int k2 = kk & 1 ? H - 1 - j0 - (kk >> 1) : H + j0 + (kk >> 1);
            const int i = (line * P.P + k2) * P.P + k3;
            if (k2 < P.P) direct_product(P, p, adjoint, i, q, Y + i * ld + q);
        }
}

// ---- adjoint -----------------------------------------------------------------
//
// grad(p) = sum over k' - h = p of (Z W^T)[k', h], Z[k'] = sum_l (U gS_l Sigma^{-1})[k' - e_l],
// W = conj(V) (adjoint.hip). Per frequency of the axes 2..d
//     Z~_w[k1'] = sum_i U~_w[k1' - 1, i] G_1[i] + U~_w[k1', i] sum_{l >= 2} e^{-2 pi i w_l / L} G_l[i],
//     g~_w(p1)  = sum over k1' - h1 = p1 of Z~_w[k1'] . conj(V~_w[h1]),
// G_l = gS_l Sigma^{-1}, and grad is the inverse transform of g~. U~ and V~ are those of the
// S-build: the phase of their lines' centres cancels in U~ conj(V~). d >= 2 only; d = 1 keeps
// the tiles of adjoint.hip (points of two folded lines would fall on one sample).
//   8 (n+2)(n+1) m L^(d-1) operations instead of 8 (n+2)^d (n+1)^d m; pack, tiles and sums
// against the three launches here, in us: d=2 n=15 m=8 17.3 -> 15.9, d=2 n=63 m=20 137 -> 42,
// d=3 n=12 m=11 63 -> 25, d=3 n=15 m=17 104 -> 38. What is left is latency: the loads of a
// unit's U~ and V~ (spectral_adjoint 17 us at d=2 n=63, 3 us of it matrix work) and the
// transforms' short chains.

struct SpecAdjPtrs {
    SpecPtrs p;          // U, V and their transforms, sigma, tab
    const double2* gS;
    double2* gt;         // g~[w][t]; d = 2: by 16-row block of k1', [block][w][t]
    double2* gf;
};

// LDS of spectral_adjoint: G [l][i][q] (padded), then per wave a 16 x 17 tile and the
// diagonal sums of a row block (d = 2) or of all of them.
__host__ __device__ inline size_t adj_g_bytes(int d, int m) {
    return 16 * (size_t)d * ((m + 3) & ~3) * (16 * ((m + 15) >> 4));
}
__host__ __device__ inline int adj_sums(int d, int K1) {
    return ((K1 + 15) & ~15) + 16 + (d == 3 ? (K1 + 16) & ~15 : 16);
}
__host__ __device__ inline size_t adj_wave_bytes(int d, int K1) { return 16 * (size_t)(16 * 17 + adj_sums(d, K1)); }

// LDS accesses of a wave before and after stay in this order (the hardware keeps it; this
// is for the compiler).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One unit, a frequency (d = 2: and a 16-row block kb of k1', for there are few frequencies;
// the blocks' sums are added where they are read), per wave and turn. Z~^T = G^T U~^T
// (rows q, columns k1') stays in registers: its result layout is the second operand's
// layout of the products conj(V~) Z~^T (rows h1), whose diagonals are summed through LDS.
template <int NQB>
__device__ __forceinline__ void adjoint_body(const SpecPlan& P, const SpecAdjPtrs& a, int wg, int wgs,
                                             unsigned char* smem) {
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = P.m, K1 = P.K1, KM = (m + 3) >> 2, MI = 4 * KM, d = P.d;
    const int nkb = (K1 + 16) >> 4, nhb = (K1 + 15) >> 4;
    constexpr int MQ = 16 * NQB;
    double2* G = reinterpret_cast<double2*>(smem);
    double2* tile = reinterpret_cast<double2*>(smem + adj_g_bytes(d, m) + adj_wave_bytes(d, K1) * wave);
    double* sums = reinterpret_cast<double*>(tile + 16 * 17);
    const double2* roots = a.p.tab + table_sizes(P.P).off_r;
    for (int e = tid; e < d * MI * MQ; e += kThreads) {
        const int q = e % MQ, i = e / MQ % MI, l = e / (MQ * MI);
        double2 v = make_double2(0.0, 0.0);
        if (q < m && i < m) {
            v = a.gS[((size_t)l * m + i) * m + q];
            const double s = a.p.sigma[q];
            v = make_double2(v.x / s, v.y / s);
        }
        G[e] = v;
    }
    __syncthreads();
    const int row_bytes = 16 * m;
    const int parts = d == 2 ? nkb : 1, sn = adj_sums(d, K1);
    for (int u = wg * kWaves + wave; u < P.F * parts; u += wgs * kWaves) {
        const int w = u / parts, part = u - w * parts;
        const auto ut = buffer_of(a.p.ut + (size_t)w * K1 * m, K1 * row_bytes);
        const auto vt = buffer_of(a.p.vt + (size_t)w * K1 * m, K1 * row_bytes);
        wave_order();
        for (int x = lane; x < 2 * sn; x += 64) sums[x] = 0.0;
        // phases e^{-2 pi i w_l / L} of the axes 2 (and 3)
        const double2 r2 = roots[d == 3 ? w / P.L : w], r3 = roots[d == 3 ? w % P.L : 0];
        for (int kb = part; kb < (d == 2 ? part + 1 : nkb); ++kb) {
            double2 zs[NQB][4];           // Z~ of column k1' = 16 kb + col, rows q = 16 qb + g + 4 r
            {
                acc_t z[NQB][3];
#pragma unroll
                for (int b = 0; b < NQB; ++b)
#pragma unroll
                    for (int x = 0; x < 3; ++x) z[b][x] = acc_t{0, 0, 0, 0};
                const int k1 = 16 * kb + col;
                for (int s0 = 0; s0 < KM; s0 += 4) {
                    double2 u0[4], u1[4];           // U~[k1'][i], U~[k1' - 1][i], i = 4 s + g
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = 4 * (s0 + k) + g, o = i < m ? k1 * row_bytes + 16 * i : kOutside;
                        u0[k] = buffer_load(ut, o);
                        u1[k] = buffer_load(ut, i < m ? o - row_bytes : kOutside);
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (s0 + k >= KM) break;
                        const double2* gi = G + (4 * (s0 + k) + g) * MQ + col;
#pragma unroll
                        for (int b = 0; b < NQB; ++b) {
                            const double2 g1 = gi[16 * b], g2 = gi[(size_t)MI * MQ + 16 * b];
                            double2 gm = make_double2(fma(r2.x, g2.x, r2.y * g2.y), fma(r2.x, g2.y, -r2.y * g2.x));
                            if (d == 3) {
                                const double2 g3 = gi[(size_t)2 * MI * MQ + 16 * b];
                                gm.x = fma(r3.x, g3.x, fma(r3.y, g3.y, gm.x));
                                gm.y = fma(r3.x, g3.y, fma(-r3.y, g3.x, gm.y));
                            }
                            z[b][0] = M::fma(g1.x, u1[k].x, z[b][0]);
                            z[b][1] = M::fma(g1.y, u1[k].y, z[b][1]);
                            z[b][2] = M::fma(g1.x + g1.y, u1[k].x + u1[k].y, z[b][2]);
                            z[b][0] = M::fma(gm.x, u0[k].x, z[b][0]);
                            z[b][1] = M::fma(gm.y, u0[k].y, z[b][1]);
                            z[b][2] = M::fma(gm.x + gm.y, u0[k].x + u0[k].y, z[b][2]);
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < NQB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        zs[b][r] = make_double2(z[b][0][r] - z[b][1][r], z[b][2][r] - z[b][0][r] - z[b][1][r]);
            }
            for (int hb = 0; hb < nhb; ++hb) {
                double2 v[NQB][4];               // V~[h1][q], h1 = 16 hb + col, q = 16 b + 4 s + g
#pragma unroll
                for (int b = 0; b < NQB; ++b)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int q = 16 * b + 4 * s + g;
                        v[b][s] = buffer_load(vt, q < m ? (16 * hb + col) * row_bytes + 16 * q : kOutside);
                    }
                acc_t x1 = {0, 0, 0, 0}, x2 = {0, 0, 0, 0}, x3 = {0, 0, 0, 0};
#pragma unroll
                for (int b = 0; b < NQB; ++b)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        if (16 * b + 4 * s >= m) break;
                        x1 = M::fma(v[b][s].x, zs[b][s].x, x1);
                        x2 = M::fma(v[b][s].y, zs[b][s].y, x2);
                        x3 = M::fma(v[b][s].x - v[b][s].y, zs[b][s].x + zs[b][s].y, x3);
                    }
                // conj(v) z at (h1 = row, k1' = col); rows past K1 are zero rows
                wave_order();
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    tile[M::row(g, r) * 17 + col] = make_double2(x1[r] + x2[r], x3[r] - x1[r] + x2[r]);
                wave_order();
                // lane 2 e + comp sums the diagonal k - h = e - 15
                const int e = lane >> 1;
                if (e < 31) {
                    const double* t = reinterpret_cast<const double*>(tile) + (lane & 1);
                    const int h0 = max(0, 15 - e), h1 = min(15, 30 - e);
                    double sum = 0.0;
#pragma unroll
                    for (int h = 0; h < 16; ++h) {
                        const double y = t[2 * (min(max(h, h0), h1) * 17 + e - 15 + min(max(h, h0), h1))];
                        sum += h >= h0 && h <= h1 ? y : 0.0;
                    }
                    // t = k1' - h1 + K1 - 1: place 16 (kb - part + nhb - hb) + e - 15
                    // holds t = 16 part + K1 - 1 - 16 nhb + place
                    sums[2 * (16 * (kb - part + nhb - hb) + e - 15) + (lane & 1)] += sum;
                }
                wave_order();
            }
        }
        const int t0 = 16 * part + K1 - 1 - 16 * nhb, t1 = d == 2 ? 16 * part + 14 + K1 : P.NP1 - 1;
        double2* out = a.gt + ((size_t)part * P.F + w) * P.NP1;
        for (int x = lane; x < sn; x += 64) {
            const int t = t0 + x;
            if (t >= 16 * part && t <= t1 && t < P.NP1) out[t] = make_double2(sums[2 * x], sums[2 * x + 1]);
        }
    }
}

// g~ at frequencies w and -w (d = 2), summed over the row blocks that reach t (in order).
__device__ __forceinline__ void adjoint_pair(const SpecPlan& P, const double2* __restrict__ gt, int w, int t,
                                             double2& x, double2& y) {
    const int nkb = (P.K1 + 16) >> 4, hi = min(nkb - 1, t >> 4);
    const bool two = w > 0 && w < P.P;
    x = y = make_double2(0.0, 0.0);
    constexpr int kIn = 4;
    for (int kb = max(0, (t - P.K1 + 1) >> 4); kb <= hi; kb += kIn) {
        double2 a[kIn], b[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const double2* g = gt + (size_t)(kb + k) * P.F * P.NP1 + t;
            a[k] = kb + k <= hi ? g[(size_t)w * P.NP1] : make_double2(0.0, 0.0);
            b[k] = kb + k <= hi && two ? g[(size_t)(P.L - w) * P.NP1] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            x = make_double2(x.x + a[k].x, x.y + a[k].y);
            y = make_double2(y.x + b[k].x, y.y + b[k].y);
        }
    }
}

// Writes component `im` of grad(p) and returns whether it is not finite. Points with two
// coordinates n + 1, and the point with all coordinates -n, belong to no T_l.
__device__ __forceinline__ bool store_gradient(const SpecPlan& P, const SpecAdjPtrs& a, const int (&p)[3], bool im,
                                               double x) {
    const int top = P.n + 1, low = -P.n;
    if ((p[0] == top) + (p[1] == top) + (P.d == 3 && p[2] == top) > 1 ||
        (p[0] == low && p[1] == low && (P.d == 2 || p[2] == low)))
        x = 0.0;
    int64_t at = (int64_t)(p[0] + P.n) * P.L + p[1] + P.n;
    if (P.d == 3) at = at * P.L + p[2] + P.n;
    reinterpret_cast<double*>(a.gf + at)[im] = x;
    return !is_finite(x);
}

// The gradient's line (p1[, p2], .) from the inputs, by the whole workgroup, where its values
// are not finite (see above): per kDirect columns q and pair of lines k_o - h_o = p_o, Z
// (formed once for all points of the line) and V through LDS, a thread per point. A point
// costs its n m terms per pair, and Z d m^2 per row and pair: d = 2, n = 63, m = 20 with one
// entry of U not finite (every line at once) takes 24 ms, d = 3, n = 12, m = 11 11 ms. (A thread
// per point that forms Z anew for each of its terms takes m^2 steps where this takes about m,
// up to eight points one after another: 10^9 of them at d = 2, n = 239, m = 32.)
constexpr int kDirect = 4;
__host__ __device__ inline size_t direct_bytes(int d, int n, int m) {
    return sizeof(double2) * kDirect * (2 * (size_t)(n + 2) + d * m);
}
__device__ __forceinline__ void direct_line(const SpecPlan& P, const SpecAdjPtrs& a, int p1, int p2,
                                            unsigned char* smem) {
    // (opaque, so that nothing of this rare path is computed before it is taken)
    int n = P.n, m = P.m;
    asm volatile("" : "+s"(n), "+s"(m));
    const int d = P.d, E = n + 1, tid = threadIdx.x;
    double2* zs = reinterpret_cast<double2*>(smem);          // [k][kDirect], k <= n + 1
    double2* vs = zs + (size_t)(n + 2) * kDirect;            // conj V, [h][kDirect]
    double2* gs = vs + (size_t)(n + 2) * kDirect;            // gS_l Sigma^{-1}, [l][i][kDirect]
    double2* g = a.gf + (d == 3 ? (int64_t)(p1 + n) * P.L + p2 + n : p1 + n) * P.L;
    constexpr int kOwn = 2;                                  // 2 n + 2 <= 480 points
    double2 sum[kOwn];
    unsigned bad = 0;                                        // bits 2 x, 2 x + 1: point x's components
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
        sum[x] = make_double2(0.0, 0.0);
        const int at = tid + kThreads * x;
        if (at < P.L) bad |= (is_finite(g[at].x) ? 0u : 1u << 2 * x) | (is_finite(g[at].y) ? 0u : 2u << 2 * x);
    }
    const int n2 = d == 3 ? min(n + 1, n + p2) - max(0, p2) + 1 : 1;         // lines of axis 2 that meet
    const int pairs = (min(n + 1, n + p1) - max(0, p1) + 1) * n2;
    for (int x = 0; x < pairs * ((m + kDirect - 1) / kDirect); ++x) {
        // done where every sum wanted is NaN
        bool open = false;
#pragma unroll
        for (int y = 0; y < kOwn; ++y)
            open |= ((bad >> 2 * y & 1) && sum[y].x == sum[y].x) || ((bad >> 2 * y & 2) && sum[y].y == sum[y].y);
        if (!__syncthreads_or(open)) break;
        const int q0 = x / pairs * kDirect, pair = x % pairs;
        if (pair == 0) {
            for (int e = tid; e < d * m * kDirect; e += kThreads) {
                const int q = min(q0 + e % kDirect, m - 1);
                const double2 w = a.gS[(size_t)(e / kDirect) * m + q];
                gs[e] = make_double2(w.x / a.p.sigma[q], w.y / a.p.sigma[q]);
            }
            __syncthreads();
        }
        const int k1 = max(0, p1) + pair / n2, k2 = d == 3 ? max(0, p2) + pair % n2 : 0;
        if (k1 == n + 1 && k2 == n + 1) continue;            // rows of no T_l
        // rows that some T_l holds: not the origin, one coordinate n + 1 at most
        const int lo = k1 + k2 == 0 ? 1 : 0, hi = k1 == n + 1 || k2 == n + 1 ? n : n + 1;
        const int64_t vrow = (int64_t)(d == 3 ? (k1 - p1) * E + k2 - p2 : k1 - p1) * E;
        for (int e = tid; e < (n + 2) * kDirect; e += kThreads) {
            const int k = e / kDirect, q = q0 + e % kDirect;
            double2 z = make_double2(0.0, 0.0), v = z;
            if (k >= lo && k <= hi && q < m)
                for (int l = 0; l < d; ++l) {
                    const int c[3] = {k1, d == 3 ? k2 : k, k};
                    bool inside = true;
                    int row = 0;
                    for (int axis = 0; axis < d; ++axis) {
                        const int y = c[axis] - (axis == l ? 1 : 0);
                        inside = inside && y >= 0 && y <= n;
                        row = row * E + y;
                    }
                    if (!inside) continue;
#pragma unroll 8
                    for (int i = 0; i < m; ++i) {
                        const double2 u = a.p.U[row * a.p.u_rs + i * a.p.u_cs];
                        const double2 w = gs[(l * m + i) * kDirect + e % kDirect];
                        z.x = fma(u.x, w.x, fma(-u.y, w.y, z.x));
                        z.y = fma(u.x, w.y, fma(u.y, w.x, z.y));
                    }
                }
            if (k <= n && q < m) v = a.p.V[(vrow + k) * a.p.v_rs + q * a.p.v_cs];
            zs[e] = z;
            vs[e] = make_double2(v.x, -v.y);
        }
        __syncthreads();
#pragma unroll
        for (int y = 0; y < kOwn; ++y) {
            const int p = tid + kThreads * y - n;
            if (!(bad >> 2 * y & 3)) continue;
            const int h1 = min(n, hi - p);
#pragma unroll 2
            for (int h = max(0, lo - p); h <= h1; ++h) {
                double2 t = make_double2(0.0, 0.0);
#pragma unroll
                for (int c = 0; c < kDirect; ++c) {
                    const double2 z = zs[(h + p) * kDirect + c], v = vs[h * kDirect + c];
                    t.x = fma(z.x, v.x, fma(-z.y, v.y, t.x));
                    t.y = fma(z.x, v.y, fma(z.y, v.x, t.y));
                }
                sum[y].x += t.x;
                sum[y].y += t.y;
            }
        }
    }
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
        const int at = tid + kThreads * x;
        if (bad >> 2 * x & 1) g[at].x = sum[x].x;
        if (bad >> 2 * x & 2) g[at].y = sum[x].y;
    }
    __syncthreads();
}

// Inverse transform of g~ at the points +-j, j = 0..P, of a transformed axis: C +- S with
// A = g~(w) + g~(-w), i B over w = 0..P (w = 0 and P alone, no sine part); the factors are
// those of the sample grid's forward transform with rows and contraction exchanged.
// d = 2: 8 sample lines per workgroup.
__device__ __forceinline__ void adjoint_lines(const SpecPlan& P, const SpecAdjPtrs& a, int blk, unsigned char* smem) {
    __shared__ int bad_flag;
    if (threadIdx.x == 0) bad_flag = 0;
    const TableSizes T = table_sizes(P.P);
    const int K = P.P + 1, KS = T.ks_g, J = line_rows(K);
    double2* xc = reinterpret_cast<double2*>(smem);
    double2* xi = xc + (size_t)J * kCols;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < J * kCols; e += kThreads) {
        const int t = kCols * blk + (e & 7), w = e >> 3;
        double2 x = make_double2(0.0, 0.0), y = x;
        if (t < P.NP1 && w < K) adjoint_pair(P, a.gt, w, t, x, y);
        xc[e] = make_double2(x.x + y.x, x.y + y.y);
        xi[e] = make_double2(y.y - x.y, x.x - y.x);
    }
    __syncthreads();
    const double scale = 1.0 / P.F;
    bool bad = false;
    for (int rb = wave; 16 * rb < K; rb += kWaves) {
        const double2* f = a.p.tab + T.off_g + (size_t)rb * KS * 64 + lane;
        const double* x1 = reinterpret_cast<const double*>(xc) + 16 * g + col;
        const double* x2 = reinterpret_cast<const double*>(xi) + 16 * g + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        for (int s = 0; s < KS; s += 4)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (s + k >= KS) break;
                const double2 t = f[64 * (s + k)];
                ac = M::fma(t.x, x1[64 * (s + k)], ac);
                as = M::fma(t.y, x2[64 * (s + k)], as);
            }
        const int t = kCols * blk + (col >> 1);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int j = 16 * rb + M::row(g, r >> 1);
            const double x = (r & 1 ? ac[r >> 1] - as[r >> 1] : ac[r >> 1] + as[r >> 1]) * scale;
            const int pt[3] = {t - P.n, r & 1 ? -j : j, 0};
            if (t < P.NP1 && j < K && (!(r & 1) || (j > 0 && j < P.P))) bad |= store_gradient(P, a, pt, col & 1, x);
        }
    }
    if (__builtin_expect(any_bad(bad, &bad_flag), 0))
        for (int t = kCols * blk; t < min(kCols * (blk + 1), P.NP1); ++t) direct_line(P, a, t - P.n, 0, smem);
}

// d = 3: the points +-j of axis 2, j in part `split`, of sample line t: axis 2 into LDS
// as the operands of axis 3's pairs u = 0..P, then axis 3.
__device__ __forceinline__ void adjoint_planes(const SpecPlan& P, const SpecAdjPtrs& a, int t, int split,
                                               unsigned char* smem) {
    __shared__ int bad_flag;
    if (threadIdx.x == 0) bad_flag = 0;
    const TableSizes T = table_sizes(P.P);
    const int K = P.P + 1, KS = T.ks_g;
    const int j0 = split * P.irows, kn = min(P.irows, K - j0);
    const int ts = plane_stride(2 * P.irows);
    double* tc = reinterpret_cast<double*>(smem);       // [u][2 j + side], A
    double* ti = tc + (size_t)4 * KS * ts;              // i B
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool odd = lane & 1;
    for (int i = tid; i < (4 * KS - K) * ts; i += kThreads) {
        tc[(size_t)K * ts + i] = 0.0;
        ti[(size_t)K * ts + i] = 0.0;
    }
    const double2* tab = a.p.tab + T.off_g;
    const int jr = min(j0 + col, K - 1);
    const double2* tab2 = tab + (size_t)(jr >> 4) * KS * 64 + 16 * g + (jr & 15);
    for (int it = wave; 8 * it < K; it += kWaves) {
        const int u = 8 * it + (col >> 1);
        acc_t ac[2], as[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) ac[i] = as[i] = acc_t{0, 0, 0, 0};
        constexpr int kIn = 4;
        for (int s0 = 0; s0 < KS; s0 += kIn) {
            double2 f[kIn], x[2][kIn], y[2][kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                f[k] = tab2[64 * (s0 + k)];
                const int w = 4 * (s0 + k) + g;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const bool in = u < K && w < K && (i == 0 || (u > 0 && u < P.P));
                    const double2* g3 = a.gt + (size_t)(i == 0 ? u : P.L - u) * P.NP1 + t;
                    const size_t step = (size_t)P.L * P.NP1;
                    x[i][k] = in ? g3[w * step] : make_double2(0.0, 0.0);
                    y[i][k] = in && w > 0 && w < P.P ? g3[(P.L - w) * step] : make_double2(0.0, 0.0);
                }
            }
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                if (s0 + k >= KS) break;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    // A, and i B
                    const double2 p = x[i][k], q = y[i][k];
                    ac[i] = M::fma(f[k].x, odd ? p.y + q.y : p.x + q.x, ac[i]);
                    as[i] = M::fma(f[k].y, odd ? p.x - q.x : q.y - p.y, as[i]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = M::row(g, r);
#pragma unroll
            for (int h = 0; h < 2; ++h) {               // the points +j and -j
                const double x = h == 0 ? ac[0][r] + as[0][r] : ac[0][r] - as[0][r];
                const double y = h == 0 ? ac[1][r] + as[1][r] : ac[1][r] - as[1][r];
                const double b = swap_lane_pair(x - y);
                if (u < K && j < kn) {
                    tc[u * ts + 2 * (2 * j + h) + (col & 1)] = x + y;
                    ti[u * ts + 2 * (2 * j + h) + (col & 1)] = odd ? b : -b;
                }
            }
        }
    }
    __syncthreads();
    const int nc2 = 2 * kn, nb2 = (nc2 + 7) >> 3, nrb = (K + 15) >> 4;
    const double scale = 1.0 / P.F;
    bool bad = false;
    for (int it = wave; it < nb2 * nrb; it += kWaves) {
        const int nb = it / nrb, rb = it - nb * nrb;
        const double2* f = tab + (size_t)rb * KS * 64 + lane;
        const double* x1 = tc + g * ts + 16 * nb + col;
        const double* x2 = ti + g * ts + 16 * nb + col;
        acc_t ac = {0, 0, 0, 0}, as = {0, 0, 0, 0};
        for (int s = 0; s < KS; ++s) {
            const double2 c = f[64 * s];
            ac = M::fma(c.x, x1[4 * s * ts], ac);
            as = M::fma(c.y, x2[4 * s * ts], as);
        }
        const int c = 8 * nb + (col >> 1), j2 = j0 + (c >> 1);
        const bool mirror = c & 1;
        const int p2 = mirror ? -j2 : j2;
        const bool ok = c < nc2 && (!mirror || (j2 > 0 && j2 < P.P));
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int j = 16 * rb + M::row(g, r >> 1);
            const double x = (r & 1 ? ac[r >> 1] - as[r >> 1] : ac[r >> 1] + as[r >> 1]) * scale;
            const int pt[3] = {t - P.n, p2, r & 1 ? -j : j};
            if (ok && j < K && (!(r & 1) || (j > 0 && j < P.P))) bad |= store_gradient(P, a, pt, col & 1, x);
        }
    }
    if (__builtin_expect(any_bad(bad, &bad_flag), 0))
        for (int c = 0; c < 2 * kn; ++c) {
            const int j2 = j0 + (c >> 1);
            if (!(c & 1) || (j2 > 0 && j2 < P.P)) direct_line(P, a, t - P.n, c & 1 ? -j2 : j2, smem);
        }
}

template <int NQB>
__global__ __launch_bounds__(kThreads) void spectral_adjoint(SpecPlan P, SpecAdjPtrs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    adjoint_body<NQB>(P, a, blockIdx.x, gridDim.x, smem);
}

__global__ __launch_bounds__(kThreads) void spectral_adjoint_inverse(SpecPlan P, SpecAdjPtrs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (P.d == 2)
        adjoint_lines(P, a, blockIdx.x, smem);
    else
        adjoint_planes(P, a, blockIdx.x / P.isplits, blockIdx.x % P.isplits, smem);
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
bool plan_forward(prony_handle_t h, int d, int n, int m, SpecPlan& P, bool batched = false) {
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
    P.npb = (P.P + 15) / 16;
    P.nqb = (m + 15) / 16;
    const size_t budget = lds_budget(h);
    // LDS that a block count is chosen for: members of a batch share their launch, whose
    // workgroups all take the LDS of the largest (96 uneven instances: 56 us with 72 KB,
    // 47.5 with 54 KB, 48 with 40 KB, 50 with 27 KB)
    const size_t want = batched ? std::min<size_t>(budget, 40960) : budget;
    if (d <= 2) {
        // column blocks per workgroup so that its items (a block of pairs against up to two
        // column blocks) occupy the four waves
        P.nbw = P.npb == 1 ? 8 : P.npb <= 3 ? 8 / (P.npb + (P.npb & 1)) : P.npb == 4 ? 1 : 2;
        auto lds = [&](int nb, bool grid) {
            return 2 * 16 * kCols * (size_t)nb * line_rows(folded_points(P.P, grid));
        };
        while (P.nbw > 1 && lds(P.nbw, false) > want) --P.nbw;
        P.nbwf = P.nbw;
        while (P.nbwf > 1 && lds(P.nbwf, true) > want) --P.nbwf;
        auto wgs = [&](int64_t cols, int nb) { return (int)(((cols + kCols - 1) / kCols + nb - 1) / nb); };
        // a single instance takes narrower workgroups rather than leave half the CUs idle
        auto count = [&](int nb, int nbf) { return 2 * wgs((int64_t)P.K1 * m, nb) + wgs(P.NP1, nbf); };
        while (!batched && P.nbw > 1 && 2 * count((P.nbw + 1) / 2, P.nbwf) <= h->num_cus) P.nbw = (P.nbw + 1) / 2;
        while (!batched && P.nbwf > 1 && 2 * count(P.nbw, (P.nbwf + 1) / 2) <= h->num_cus) P.nbwf = (P.nbwf + 1) / 2;
        P.lds_fwd = std::max(lds(P.nbw, false), lds(P.nbwf, true));
        P.wgs_x = wgs((int64_t)P.K1 * m, P.nbw);
        P.wgs_f = wgs(P.NP1, P.nbwf);
    } else {
        // a workgroup takes one block of 16 pairs of axis 3 and as many columns as fit
        auto lds = [&](int nq, int J) { return 8 * (size_t)(J + 1) * plane_stride(2 * std::min(P.P, 16) * nq); };
        for (P.nq = std::min(m, kCols); P.nq > 0; P.nq /= 2) {
            P.lds_fwd = std::max(lds(P.nq, P.P), lds(1, P.L));
            if (P.lds_fwd <= (P.nq > 1 ? want : budget)) break;
        }
        if (P.nq == 0) return false;
        // a single instance takes narrower workgroups rather than leave half the CUs idle
        auto count = [&](int nq) { return (2 * P.K1 * ((m + nq - 1) / nq) + P.NP1) * P.npb; };
        while (!batched && P.nq > 2 && 2 * count(P.nq) <= h->num_cus) P.nq /= 2;
        P.splits = P.npb;
        P.wgs_x = P.K1 * ((m + P.nq - 1) / P.nq) * P.splits;
        P.wgs_f = P.NP1 * P.splits;
    }
    return P.lds_fwd <= budget;
}

constexpr size_t kMaxWorkspace = size_t(1) << 30;
// A batch's memory, once for S and once for gradients: two to four times what its tiles need
// (d = 3, n = 15, m = 32: 26 MB an instance against 12), so past about a quarter of the
// card's memory the rest is left to the caller.
constexpr size_t kMaxBatch = size_t(64) << 30;
constexpr size_t kMaxTables = size_t(64) << 20;

void fill_tables(prony_handle_t h, int P, double2* tab) {
    const int blocks = (table_sizes(P).total + kThreads - 1) / kThreads;
    spectral_fill_tables<<<std::min(blocks, 4 * h->num_cus), kThreads, 0, h->stream>>>(P, tab);
}

// The tables of lines of P points: kept by the handle from the first call that needs them
// (at most kMaxTables in all), else made on each call at `ws`, the plan's workspace
// section (without `keep`, under stream capture, where nothing can be allocated, or past
// the limit). Calls of one handle on several streams are ordered (prony_set_stream).
prony_status_t tables_for(prony_handle_t h, int P, double2* ws, bool keep, const double2** tab) {
    const auto it = h->spectral_tables.find(P);
    if (it != h->spectral_tables.end()) {
        *tab = static_cast<const double2*>(it->second);
        return PRONY_OK;
    }
    const size_t bytes = 16 * (size_t)table_sizes(P).total;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(h->stream, &cs);
    if (e != hipSuccess) return hip_fail(h, e, "hipStreamIsCapturing");
    void* mem = nullptr;
    if (keep && cs == hipStreamCaptureStatusNone && h->spectral_table_bytes + bytes <= kMaxTables &&
        hipMalloc(&mem, bytes) == hipSuccess) {
        h->spectral_tables[P] = mem;
        h->spectral_table_bytes += bytes;
        ws = static_cast<double2*>(mem);
    } else {
        (void)hipGetLastError();
    }
    *tab = ws;
    if (!ws) return PRONY_OK;
    fill_tables(h, P, ws);
    return check_launch(h, "spectral_fill_tables");
}

}  // namespace

prony_status_t spectral_reserve(prony_handle_t h, int d_max, int n_max) {
    for (int n = 1; n <= n_max; ++n)
        for (int d = 1; d <= std::min(d_max, 2); ++d) {     // d = 3 has the lines of d = 2
            SpecPlan P;
            if (!plan_forward(h, d, n, 1, P)) continue;
            const double2* tab = nullptr;
            const prony_status_t st = tables_for(h, P.P, nullptr, true, &tab);
            if (st != PRONY_OK) return st;
        }
    return PRONY_OK;
}

size_t spectral_reserve_bytes(prony_handle_t h, int d, int n_max, int m_max) {
    size_t best = 0;
    for (int n = 1; n <= std::min(n_max, d == 1 ? kMaxLines * kMaxLines : kMaxLines); ++n) {
        const int top = (int)std::min<int64_t>(std::min(m_max, 32), ipow(n + 1, d));
        for (int m = 1; m <= top; ++m) {
            // (d = 1 stays far below the limit on the workspace: it grows with m between
            // the steps in the number of column blocks)
            if (d == 1 && m != top && m % 16) continue;
            SpecPlan P;
            if (spectral_plan(h, d, n, m, true, P)) best = std::max(best, P.ws_bytes);
            if (spectral_adjoint_plan(h, d, n, m, P)) best = std::max(best, P.ws_bytes);
        }
    }
    return best;
}

size_t spectral_table_bytes(const SpecPlan& P) { return align_up(16 * (size_t)table_sizes(P.P).total, 256); }

// Single S-builds up to here run the tiles: two launches with prepared factors instead of three
// (d=1 n=63 m=5 10.4 us against 13.4, n=255 m=8 12.2 against 13.0; d=2 n=7 m=8 11.1 against 13.0, n=15 m=5
// 13.2 either way; d=3 n=2 m=12 10.5 against 13.0, n=3 m=8 12.6 against 13.0), three without
// allocation instead of the four that make the tables as well (14.8 against 16.7 to 17.6),
// three either way in prony_build_S (14.7 to 15.2 both; d=3 n=3 15.5 against 14.7).
static bool small_build(int d, int n, int m) {
    return ipow(n + 1, d) <= (m <= 8 ? (d == 1 ? 256 : d == 2 ? 64 : 32) : m > 16 ? 0 : d == 1 ? 64 : 32);
}

bool spectral_plan(prony_handle_t h, int d, int n, int m, bool s0, SpecPlan& P, bool batched) {
    if (!batched && small_build(d, n, m)) return false;
    if (!plan_forward(h, d, n, m, P, batched)) return false;
    P.s0 = s0 ? 1 : 0;
    P.ells = d + P.s0;
    P.nmb = ((d >= 2 ? 2 * m : m) + 15) / 16;
    P.nm0 = P.nqb;
    P.ns = d == 3 || s0 ? 2 : 1;
    const int outer = d == 3 ? P.L : 1;
    // a single instance fills the GPU with two workgroups per CU; a batch member takes
    // workgroups of about 512 products of 16 x 16 x 4 whatever else the batch holds (so that
    // its results do not depend on that): batches of 8 / 30 / 96 / 250 instances take 18 / 25
    // / 96 / 284 us, with 256 products 13 / 27 / 105 / 336, with 1024 26 / 32 / 92 / 262
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
    P.ws_bytes = P.off_r + spectral_table_bytes(P);
    return P.ws_bytes <= kMaxWorkspace;
}

bool spectral_product_plan(prony_handle_t h, int d, int n, int r, SpecPlan& P) {
    if (!plan_forward(h, d, n, r, P)) return false;
    P.pmax = n;
    const size_t budget = lds_budget(h);
    const int KS = (P.P + 3) / 4, H = folded_points(P.P, false);
    if (d <= 2) {
        const int nrb = (H + 15) / 16;
        auto lds = [&](int nb) { return 2 * 16 * kCols * (size_t)nb * line_rows(P.P); };
        P.nbi = nrb == 1 ? 4 : nrb <= 3 ? 2 : 1;
        while (P.nbi > 1 && lds(P.nbi) > budget) --P.nbi;
        P.lds_inv = lds(P.nbi);
        P.wgs_i = ((P.K1 * r + kCols - 1) / kCols + P.nbi - 1) / P.nbi;
    } else {
        // at most 16 folded rows of axis 2 per workgroup, at least 4, about one workgroup per CU
        for (P.nqi = std::min(r, kCols); P.nqi > 0; P.nqi /= 2) {
            const int lines = P.K1 * ((r + P.nqi - 1) / P.nqi);
            P.isplits = std::max((H + 15) / 16, std::min((H + 3) / 4, h->num_cus / lines));
            P.irows = (H + P.isplits - 1) / P.isplits;
            P.lds_inv = 2 * 8 * (size_t)(4 * KS) * plane_stride(2 * P.irows * P.nqi);
            if (P.lds_inv <= budget) break;
        }
        if (P.nqi == 0) return false;
        P.isplits = (H + P.irows - 1) / P.irows;
        P.wgs_i = P.K1 * ((r + P.nqi - 1) / P.nqi) * P.isplits;
    }
    if (P.lds_inv > budget) return false;
    const size_t x = align_up(16 * (size_t)P.F * P.K1 * r, 256);
    P.off_v = x;
    P.off_f = 2 * x;
    P.off_r = P.off_f + align_up(16 * (size_t)P.F * P.NP1, 256);
    P.ws_bytes = P.off_r + spectral_table_bytes(P);
    return P.ws_bytes <= kMaxWorkspace;
}

bool spectral_adjoint_plan(prony_handle_t h, int d, int n, int m, SpecPlan& P, bool batched) {
    if (d == 1 || !plan_forward(h, d, n, m, P, batched)) return false;
    const size_t budget = lds_budget(h);
    P.lds_gram = adj_g_bytes(d, m) + kWaves * adj_wave_bytes(d, P.K1);
    const int nkb = d == 2 ? (P.K1 + 16) / 16 : 1;
    // a wave of a batch member takes about four units (the staging of G is per workgroup)
    const int units = kWaves * (batched ? 4 : 1);
    P.groups = (int)std::min<int64_t>(((int64_t)P.F * nkb + units - 1) / units, 4 * (int64_t)h->num_cus);
    if (d == 2) {
        P.wgs_i = (P.NP1 + kCols - 1) / kCols;
        P.lds_inv = 2 * 16 * kCols * (size_t)line_rows(P.P + 1);
    } else {
        const int K = P.P + 1;
        P.isplits = std::max((K + 15) / 16, batched ? 1 : std::min((K + 3) / 4, h->num_cus / P.NP1));
        P.irows = (K + P.isplits - 1) / P.isplits;
        P.isplits = (K + P.irows - 1) / P.irows;
        P.wgs_i = P.NP1 * P.isplits;
        P.lds_inv = 2 * 8 * (size_t)(4 * table_sizes(P.P).ks_g) * plane_stride(2 * P.irows);
    }
    P.lds_inv = std::max(P.lds_inv, direct_bytes(d, n, m));
    if (P.lds_gram > budget || P.lds_inv > budget) return false;
    const size_t x = align_up(16 * (size_t)P.F * P.K1 * m, 256);
    P.off_v = x;
    P.off_f = 2 * x;
    P.off_r = P.off_f + align_up(16 * (size_t)nkb * P.F * P.NP1, 256);
    P.ws_bytes = P.off_r + spectral_table_bytes(P);
    return P.ws_bytes <= kMaxWorkspace;
}

prony_status_t spectral_adjoint_run(prony_handle_t h, const SpecPlan& P, unsigned char* ws, const double* U,
                                    int64_t u_rs, int64_t u_cs, const double* sigma, const double* V, int64_t v_rs,
                                    int64_t v_cs, const double* gS, double* gf) {
    SpecAdjPtrs a{};
    a.p.U = reinterpret_cast<const double2*>(U);
    a.p.V = reinterpret_cast<const double2*>(V);
    a.p.u_rs = u_rs;
    a.p.u_cs = u_cs;
    a.p.v_rs = v_rs;
    a.p.v_cs = v_cs;
    a.p.sigma = sigma;
    a.p.ut = reinterpret_cast<double2*>(ws);
    a.p.vt = reinterpret_cast<double2*>(ws + P.off_v);
    a.p.tables = reinterpret_cast<double2*>(ws + P.off_r);
    a.gS = reinterpret_cast<const double2*>(gS);
    a.gt = reinterpret_cast<double2*>(ws + P.off_f);
    a.gf = reinterpret_cast<double2*>(gf);
    prony_status_t st = spectral_forward(h, P, a.p, true, false, true);
    if (st != PRONY_OK) return st;
    const bool one = P.nqb == 1;
    if ((st = one ? allow_lds(h, &spectral_adjoint<1>, P.lds_gram) : allow_lds(h, &spectral_adjoint<2>, P.lds_gram)) !=
        PRONY_OK)
        return st;
    {
        ProfileScope prof(h, "spectral_adjoint");
        if (one)
            spectral_adjoint<1><<<P.groups, kThreads, P.lds_gram, h->stream>>>(P, a);
        else
            spectral_adjoint<2><<<P.groups, kThreads, P.lds_gram, h->stream>>>(P, a);
    }
    if ((st = check_launch(h, "spectral_adjoint")) != PRONY_OK) return st;
    if ((st = allow_lds(h, &spectral_adjoint_inverse, P.lds_inv)) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_inverse");
        spectral_adjoint_inverse<<<P.wgs_i, kThreads, P.lds_inv, h->stream>>>(P, a);
    }
    return check_launch(h, "spectral_adjoint_inverse");
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
    prony_status_t st = tables_for(h, P.P, reinterpret_cast<double2*>(ws + P.off_r), true, &p.tab);
    if (st != PRONY_OK) return st;
    if ((st = allow_lds(h, &spectral_forward_kernel, P.lds_fwd)) != PRONY_OK) return st;
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
            spectral_inverse_planes<<<P.wgs_i, kThreads, P.lds_inv, h->stream>>>(P, p, y, ldy, adjoint ? 1 : 0);
        else
            spectral_inverse_lines<<<P.wgs_i, kThreads, P.lds_inv, h->stream>>>(P, p, y, ldy, adjoint ? 1 : 0);
    }
    return check_launch(h, "spectral_inverse");
}

// ---- batches -----------------------------------------------------------------

struct SpecBatch {
    void* ws = nullptr;          // entries, maps, tables, then the instances' workspaces
    // the entry of every workgroup of the forward and of the Gram launch, a slice per
    // finishing workgroup
    const int* fwd_map = nullptr;
    const int* gram_map = nullptr;
    const BatchSlice* finish = nullptr;
    int fwd_wgs = 0, gram_wgs = 0, finishes = 0;
    size_t lds_fwd = 0, lds_gram = 0;
};

namespace {

// One instance of a batch: its plan and operands, its first workgroup in the forward
// launch and in its class's Gram launch.
struct SpecEntry {
    SpecPlan P;
    SpecPtrs p;
    int fwd_begin, gram_begin;
};

// A workgroup reads its entry from a table: a binary search over the entries was seven
// loads one after another, 2 us of the 10 to 20 of a workgroup.
__global__ __launch_bounds__(kThreads) void spectral_forward_batched(const SpecEntry* __restrict__ entries,
                                                                     const int* __restrict__ map) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SpecEntry& e = entries[map[blockIdx.x]];
    forward_body(e.P, e.p, blockIdx.x - e.fwd_begin, smem);
}

// All instances in one launch, each workgroup through its instance's instantiation. A
// launch per instantiation on four streams held more small workgroups per CU (this one
// has the registers of the largest), but forking and joining the streams left the GPU idle
// for longer than the launches ran beside each other.
__global__ __launch_bounds__(kThreads, 2) void spectral_gram_batched(const SpecEntry* __restrict__ entries,
                                                                     const int* __restrict__ map) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SpecEntry& e = entries[map[blockIdx.x]];
    const int x = blockIdx.x - e.gram_begin;
    switch (e.P.nmb * 16 + e.P.nm0 * 4 + e.P.ns) {
#define PRONY_CASE(B, B0, K)                                                  \
    case B * 16 + B0 * 4 + K:                                                 \
        gram_body<B, B0, K>(e.P, e.p, x / e.P.nqb, x % e.P.nqb, smem);        \
        break;
        PRONY_GRAM_CASES(PRONY_CASE)
#undef PRONY_CASE
    }
}

__global__ __launch_bounds__(kFinishThreads) void spectral_finish_batched(const SpecEntry* __restrict__ entries,
                                                                          const BatchSlice* __restrict__ slices) {
    const BatchSlice x = slices[blockIdx.x];
    const SpecEntry& e = entries[x.entry];
    finish_body(e.P, e.p, x.block);
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
    // the largest workgroups first
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    auto work = [&](int i) {
        return (double)plans[i].F * plans[i].K1 * plans[i].m * (plans[i].K1 + 2 * plans[i].m) / plans[i].groups;
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return work(a) > work(b); });
    int64_t fwd_wgs = 0, gram_wgs = 0;
    for (const SpecPlan& P : plans) {
        fwd_wgs += P.wgs_f + 2 * (int64_t)P.wgs_x;
        gram_wgs += (int64_t)P.groups * P.nqb;
    }
    if (fwd_wgs > INT32_MAX / 4 || gram_wgs > INT32_MAX / 4)
        return fail(h, PRONY_ENOTSUP, "prony_batch_create: too many workgroups");
    std::vector<int> maps;                  // forward, then Gram
    std::vector<BatchSlice> finish;
    maps.reserve((size_t)(fwd_wgs + gram_wgs));
    for (int pos = 0; pos < count; ++pos) {
        const SpecPlan& P = plans[order[pos]];
        maps.insert(maps.end(), (size_t)P.wgs_f + 2 * (size_t)P.wgs_x, pos);
        for (int b = 0; b * kFinishOuts < P.m * P.ells * P.m; ++b) finish.push_back({pos, 0, b});
    }
    for (int pos = 0; pos < count; ++pos)
        maps.insert(maps.end(), (size_t)plans[order[pos]].groups * plans[order[pos]].nqb, pos);
    // work table, maps, the tables of every line length, the instances' sections
    const size_t off_maps = align_up(sizeof(SpecEntry) * (size_t)count, 256);
    const size_t off_finish = align_up(off_maps + sizeof(int) * maps.size(), 256);
    size_t off = align_up(off_finish + sizeof(BatchSlice) * finish.size(), 256);
    std::map<int, size_t> tables;
    for (const SpecPlan& P : plans)
        if (tables.emplace(P.P, off).second) off += align_up(16 * (size_t)table_sizes(P.P).total, 256);
    std::vector<size_t> base(count);
    for (int pos = 0; pos < count; ++pos) {
        base[pos] = off;
        off += plans[order[pos]].off_r;
    }
    if (off > kMaxBatch) return fail(h, PRONY_ENOMEM, "the line-spectral form of the batch takes too much memory");
    SpecBatch* S = new (std::nothrow) SpecBatch;
    if (!S) return fail(h, PRONY_ENOMEM, "prony_batch_create: out of host memory");
    hipError_t e = hipMalloc(&S->ws, off);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete S;
        return fail(h, PRONY_ENOMEM, std::string("batch workspace allocation failed: ") + hipGetErrorString(e));
    }
    unsigned char* const ws = static_cast<unsigned char*>(S->ws);
    S->fwd_map = reinterpret_cast<const int*>(ws + off_maps);
    S->gram_map = S->fwd_map + fwd_wgs;
    S->finish = reinterpret_cast<const BatchSlice*>(ws + off_finish);
    S->fwd_wgs = (int)fwd_wgs;
    S->gram_wgs = (int)gram_wgs;
    S->finishes = (int)finish.size();
    std::vector<SpecEntry> host(count);
    int fwd = 0, wgs = 0;
    for (int pos = 0; pos < count; ++pos) {
        const int i = order[pos];
        const SpecPlan& P = plans[i];
        const prony_instance_t& x = inst[i];
        unsigned char* w = ws + base[pos];
        SpecEntry& E = host[pos];
        E.P = P;
        E.p = SpecPtrs{reinterpret_cast<const double2*>(x.U), reinterpret_cast<const double2*>(x.V), x.m, 1, x.m, 1,
                       reinterpret_cast<const double2*>(x.f), x.sigma, reinterpret_cast<double2*>(w),
                       reinterpret_cast<double2*>(w + P.off_v), reinterpret_cast<double2*>(w + P.off_f),
                       reinterpret_cast<double2*>(w + P.off_p), reinterpret_cast<double2*>(x.S), nullptr,
                       reinterpret_cast<const double2*>(ws + tables[P.P])};
        E.fwd_begin = fwd;
        fwd += P.wgs_f + 2 * P.wgs_x;
        E.gram_begin = wgs;
        wgs += P.groups * P.nqb;
        S->lds_gram = std::max(S->lds_gram, P.lds_gram);
        S->lds_fwd = std::max(S->lds_fwd, P.lds_fwd);
    }
    for (const auto& t : tables)
        fill_tables(h, t.first, reinterpret_cast<double2*>(ws + t.second));
    e = hipGetLastError();
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws, host.data(), sizeof(SpecEntry) * (size_t)count, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws + off_maps, maps.data(), sizeof(int) * maps.size(), hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws + off_finish, finish.data(), sizeof(BatchSlice) * finish.size(), hipMemcpyHostToDevice,
                           h->stream);
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
        spectral_forward_batched<<<S->fwd_wgs, kThreads, S->lds_fwd, h->stream>>>(entries, S->fwd_map);
    }
    if ((st = check_launch(h, "spectral_forward_batched")) != PRONY_OK) return st;
    if ((st = allow_lds(h, &spectral_gram_batched, S->lds_gram)) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_gram");
        spectral_gram_batched<<<S->gram_wgs, kThreads, S->lds_gram, h->stream>>>(entries, S->gram_map);
    }
    if ((st = check_launch(h, "spectral_gram_batched")) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "pencil_finish");
        spectral_finish_batched<<<S->finishes, kFinishThreads, 0, h->stream>>>(entries, S->finish);
    }
    return check_launch(h, "spectral_finish_batched");
}

// ---- batched adjoints --------------------------------------------------------

struct SpecAdjBatch {
    void* ws = nullptr;          // entries, maps, tables, then the instances' workspaces
    const int *fwd_map = nullptr, *adj_map = nullptr, *inv_map = nullptr;   // entry of every workgroup
    int fwd_wgs = 0, inv_wgs = 0;
    size_t lds_fwd = 0, lds_inv = 0;
    struct ClassLaunch {
        int nqb, first, wgs;     // first workgroup in adj_map
        size_t lds;
    };
    std::vector<ClassLaunch> launches;
};

namespace {

struct SpecAdjEntry {
    SpecPlan P;
    SpecAdjPtrs a;               // gS and gf from the call
    int64_t gs_off, gf_off;
    int fwd_begin, adj_begin, inv_begin;
};

__global__ __launch_bounds__(kThreads) void spectral_adjoint_forward_batched(const SpecAdjEntry* __restrict__ entries,
                                                                             const int* __restrict__ map) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SpecAdjEntry& e = entries[map[blockIdx.x]];
    forward_body(e.P, e.a.p, blockIdx.x - e.fwd_begin + e.P.wgs_f, smem);
}

template <int NQB>
__global__ __launch_bounds__(kThreads) void spectral_adjoint_batched(const SpecAdjEntry* __restrict__ entries,
                                                                     const int* __restrict__ map, int first,
                                                                     const double2* __restrict__ gS) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int id = first + blockIdx.x;
    const SpecAdjEntry& e = entries[map[id]];
    SpecAdjPtrs a = e.a;
    a.gS = gS + e.gs_off;
    adjoint_body<NQB>(e.P, a, id - e.adj_begin, e.P.groups, smem);
}

__global__ __launch_bounds__(kThreads) void spectral_adjoint_inverse_batched(const SpecAdjEntry* __restrict__ entries,
                                                                             const int* __restrict__ map,
                                                                             const double2* __restrict__ gS,
                                                                             double2* __restrict__ gf) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SpecAdjEntry& e = entries[map[blockIdx.x]];
    SpecAdjPtrs a = e.a;
    a.gS = gS + e.gs_off;
    a.gf = gf + e.gf_off;
    const int x = blockIdx.x - e.inv_begin;
    if (e.P.d == 2)
        adjoint_lines(e.P, a, x, smem);
    else
        adjoint_planes(e.P, a, x / e.P.isplits, x % e.P.isplits, smem);
}

}  // namespace

prony_status_t spectral_adjoint_batch_free(SpecAdjBatch* b) {
    const prony_status_t st = b->ws && hipFree(b->ws) != hipSuccess ? PRONY_EHIP : PRONY_OK;
    delete b;
    return st;
}

prony_status_t spectral_adjoint_batch_build(prony_handle_t h, const std::vector<prony_instance_t>& inst,
                                            const std::vector<int64_t>& gs_off, const std::vector<int64_t>& gf_off,
                                            SpecAdjBatch** out) {
    const int count = (int)inst.size();
    std::vector<SpecPlan> plans(count);
    int64_t fwd_wgs = 0, adj_wgs = 0, inv_wgs = 0;
    for (int i = 0; i < count; ++i) {
        SpecPlan& P = plans[i];
        if (!spectral_adjoint_plan(h, inst[i].d, inst[i].n, inst[i].m, P, true))
            return fail(h, PRONY_ENOTSUP, "an instance does not fit the line-spectral form");
        fwd_wgs += 2 * (int64_t)P.wgs_x;
        adj_wgs += P.groups;
        inv_wgs += P.wgs_i;
    }
    if (std::max({fwd_wgs, adj_wgs, inv_wgs}) > INT32_MAX / 4)
        return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint_batched: too many workgroups");
    // classes by column blocks, the largest instances first
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return plans[a].nqb != plans[b].nqb ? plans[a].nqb > plans[b].nqb
                                            : plans[a].groups * plans[a].m > plans[b].groups * plans[b].m;
    });
    std::vector<int> maps;
    maps.reserve((size_t)(fwd_wgs + adj_wgs + inv_wgs));
    for (int pos = 0; pos < count; ++pos) maps.insert(maps.end(), 2 * (size_t)plans[order[pos]].wgs_x, pos);
    for (int pos = 0; pos < count; ++pos) maps.insert(maps.end(), (size_t)plans[order[pos]].groups, pos);
    for (int pos = 0; pos < count; ++pos) maps.insert(maps.end(), (size_t)plans[order[pos]].wgs_i, pos);
    const size_t off_maps = align_up(sizeof(SpecAdjEntry) * (size_t)count, 256);
    size_t off = align_up(off_maps + sizeof(int) * maps.size(), 256);
    std::map<int, size_t> tables;
    for (const SpecPlan& P : plans)
        if (tables.emplace(P.P, off).second) off += align_up(16 * (size_t)table_sizes(P.P).total, 256);
    std::vector<size_t> base(count);
    for (int pos = 0; pos < count; ++pos) {
        base[pos] = off;
        off += plans[order[pos]].off_r;
    }
    if (off > kMaxBatch) return fail(h, PRONY_ENOMEM, "the line-spectral form of the batch takes too much memory");
    SpecAdjBatch* S = new (std::nothrow) SpecAdjBatch;
    if (!S) return fail(h, PRONY_ENOMEM, "prony_build_S_adjoint_batched: out of host memory");
    hipError_t e = hipMalloc(&S->ws, off);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete S;
        return fail(h, PRONY_ENOMEM, std::string("batch workspace allocation failed: ") + hipGetErrorString(e));
    }
    unsigned char* const ws = static_cast<unsigned char*>(S->ws);
    S->fwd_map = reinterpret_cast<const int*>(ws + off_maps);
    S->adj_map = S->fwd_map + fwd_wgs;
    S->inv_map = S->adj_map + adj_wgs;
    S->fwd_wgs = (int)fwd_wgs;
    S->inv_wgs = (int)inv_wgs;
    std::vector<SpecAdjEntry> host(count);
    int fwd = 0, adj = 0, inv = 0;
    for (int pos = 0; pos < count; ++pos) {
        const int i = order[pos];
        const SpecPlan& P = plans[i];
        const prony_instance_t& x = inst[i];
        unsigned char* w = ws + base[pos];
        SpecAdjEntry& E = host[pos];
        E.P = P;
        E.a = SpecAdjPtrs{};
        E.a.p.U = reinterpret_cast<const double2*>(x.U);
        E.a.p.V = reinterpret_cast<const double2*>(x.V);
        E.a.p.u_rs = E.a.p.v_rs = x.m;
        E.a.p.u_cs = E.a.p.v_cs = 1;
        E.a.p.sigma = x.sigma;
        E.a.p.ut = reinterpret_cast<double2*>(w);
        E.a.p.vt = reinterpret_cast<double2*>(w + P.off_v);
        E.a.p.tab = reinterpret_cast<const double2*>(ws + tables[P.P]);
        E.a.gt = reinterpret_cast<double2*>(w + P.off_f);
        E.gs_off = gs_off[i];
        E.gf_off = gf_off[i];
        E.fwd_begin = fwd;
        E.adj_begin = adj;
        E.inv_begin = inv;
        if (pos == 0 || plans[order[pos - 1]].nqb != P.nqb) S->launches.push_back({P.nqb, adj, 0, 0});
        auto& cl = S->launches.back();
        fwd += 2 * P.wgs_x;
        adj += P.groups;
        inv += P.wgs_i;
        cl.wgs = adj - cl.first;
        cl.lds = std::max(cl.lds, P.lds_gram);
        S->lds_fwd = std::max(S->lds_fwd, P.lds_fwd);
        S->lds_inv = std::max(S->lds_inv, P.lds_inv);
    }
    for (const auto& t : tables) fill_tables(h, t.first, reinterpret_cast<double2*>(ws + t.second));
    e = hipGetLastError();
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws, host.data(), sizeof(SpecAdjEntry) * (size_t)count, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws + off_maps, maps.data(), sizeof(int) * maps.size(), hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        (void)spectral_adjoint_batch_free(S);
        return hip_fail(h, e, "batch adjoint work table upload");
    }
    *out = S;
    return PRONY_OK;
}

prony_status_t spectral_adjoint_batch_launch(prony_handle_t h, const SpecAdjBatch* S, const double* gS, double* gf) {
    const SpecAdjEntry* entries = static_cast<const SpecAdjEntry*>(S->ws);
    const double2* gs2 = reinterpret_cast<const double2*>(gS);
    prony_status_t st = allow_lds(h, &spectral_adjoint_forward_batched, S->lds_fwd);
    if (st != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_forward");
        spectral_adjoint_forward_batched<<<S->fwd_wgs, kThreads, S->lds_fwd, h->stream>>>(entries, S->fwd_map);
    }
    if ((st = check_launch(h, "spectral_adjoint_forward_batched")) != PRONY_OK) return st;
    for (const auto& cl : S->launches) {
        st = cl.nqb == 1 ? allow_lds(h, &spectral_adjoint_batched<1>, cl.lds)
                         : allow_lds(h, &spectral_adjoint_batched<2>, cl.lds);
        if (st != PRONY_OK) return st;
        {
            ProfileScope prof(h, "spectral_adjoint");
            if (cl.nqb == 1)
                spectral_adjoint_batched<1><<<cl.wgs, kThreads, cl.lds, h->stream>>>(entries, S->adj_map, cl.first, gs2);
            else
                spectral_adjoint_batched<2><<<cl.wgs, kThreads, cl.lds, h->stream>>>(entries, S->adj_map, cl.first, gs2);
        }
        if ((st = check_launch(h, "spectral_adjoint_batched")) != PRONY_OK) return st;
    }
    if ((st = allow_lds(h, &spectral_adjoint_inverse_batched, S->lds_inv)) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "spectral_inverse");
        spectral_adjoint_inverse_batched<<<S->inv_wgs, kThreads, S->lds_inv, h->stream>>>(
            entries, S->inv_map, gs2, reinterpret_cast<double2*>(gf));
    }
    return check_launch(h, "spectral_adjoint_inverse_batched");
}

// ---- single instances --------------------------------------------------------

prony_status_t spectral_forward(prony_handle_t h, const SpecPlan& P, SpecPtrs& ptr, bool factors, bool grid,
                                bool keep_tables) {
    prony_status_t st = tables_for(h, P.P, ptr.tables, keep_tables, &ptr.tab);
    if (st != PRONY_OK) return st;
    if ((st = allow_lds(h, &spectral_forward_kernel, P.lds_fwd)) != PRONY_OK) return st;
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
