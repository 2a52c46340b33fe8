// Adjoint of the pencil map f -> S_l = U^* T_l(f) V Sigma^{-1} (Sec. 1, eq.
// generateSl), with U, Sigma, V held fixed: given gS_l = dL/dS_l (PyTorch's
// convention, grad = dL/dRe + i dL/dIm), the gradient on the sample grid is
//     grad(p) = sum_l sum_{k - h + e_l = p} X_l[k, h],   X_l = U gS_l Sigma^{-1} V^*.
// With k' = k + e_l as in the forward kernel (row-extended form), all d terms are
// one product of the row-extended matrix
//     Z[k', q] = sum_l (U gS_l Sigma^{-1})[k' - e_l, q]   (k' in {0..n+1}^d; a term
//                 is zero where k' - e_l leaves I_n)          ((n+2)^d x m)
// with the conjugated factor W[h, q] = conj(V[h, q]), h in I_n:
//     grad(p) = sum_{k' - h = p} (Z W^T)[k', h],
// i.e. the (n+2)^d x N product (inner dimension m) is summed along its Toeplitz
// diagonals.
//
// adjoint_pack   forms Z (FP64, stored in T), packs W as (Re, Im) pairs,
//                writes the G(h) table and zeroes the gradient;
// adjoint_tiles  one workgroup = 64 rows k' x one chunk of h: for every block of
//                16 h the tile of Z W^T is formed on MFMA (K = m; three real
//                products per complex one: Re z Re w, Im z Im w and
//                (Re z + Im z)(Re w + Im w)), and each
//                entry is added (LDS atomics, accumulation in FP64) to the bin of
//                its diagonal in an LDS copy of the workgroup's grid window; the
//                window is then added to the gradient in FP64 (device atomics).
// The accumulation order inside a bin is not fixed: results agree to rounding,
// not bitwise, between runs.
// FP64 gradients with d >= 2, single and batched, run in line-spectral form instead
// (spectral.hip) wherever it applies, the smallest single ones line by line (adjoint_lines).
#include <algorithm>

#include "common.h"
#include "mfma.h"
#include "spectral.h"

namespace prony {
namespace {

constexpr int kWaves = 4;
constexpr int kRows = kWaves * 16;
constexpr int kThreads = kWaves * 64;
constexpr int kHBlock = 16;          // h per MFMA output block (32 real columns)

struct AdjPlan {
    int d, n, N, m;
    int NR;        // (n+2)^d row-extended rows k'
    int cp;        // complex K (m) padded to a multiple of 8
    int ksteps;    // cp / 4
    int rf, rows;  // 16-row fragments per wave, rows k' per tile (64 rf)
    int kb, kc, sk, rt, nwg, win_cap, c0, gsize;
    size_t lds_bytes;
    size_t off_z, off_w, off_g, ws_bytes;
};

// Packing works in blocks, one per workgroup and turn: section 0 (Z) four units of a
// 16-row tile and 16 columns, one per wave; section 1 (W) four 16 x 16 transposes;
// section 2 (G(h) and the cleared gradient) kAdjSpan elements.
constexpr int kAdjSpan = 2048;
__host__ __device__ inline int adj_col_blocks(const AdjPlan& P) { return (P.cp + 15) >> 4; }
__host__ __device__ inline int adj_pack_blocks(const AdjPlan& P, int section) {
    const int kbp = P.sk * P.kc;
    if (section == 0) return (P.rt * (P.rows / 16) * adj_col_blocks(P) + kWaves - 1) / kWaves;
    if (section == 1) return ((kbp + 15) / 16 * adj_col_blocks(P) + 3) / 4;
    return ((kbp > P.gsize ? kbp : P.gsize) + kAdjSpan - 1) / kAdjSpan;
}

// Z is a contraction over i (K = m per matrix l) and runs on the FP64 matrix cores: each
// entry on its own lane read m entries of U and of gS per l through the vector caches,
// 2.5 GB in all for 64 instances of d=2 n=47 m=16 and 112 us; here a wave reads a row tile
// of U and a block of gS once per K step. W is read in rows of 4 columns by 16 h and
// written in rows of 16 h (its reads were 16 bytes every row).
template <typename T>
__device__ __forceinline__ void adj_pack_body(const AdjPlan& P, const double2* __restrict__ U, int64_t u_rs,
                                              int64_t u_cs, const double* __restrict__ sigma,
                                              const double2* __restrict__ V, int64_t v_rs, int64_t v_cs,
                                              const double2* __restrict__ gS, pair_t<T>* __restrict__ zp,
                                              pair_t<T>* __restrict__ wp, int* __restrict__ gt,
                                              double2* __restrict__ gf, int section, int block, int nblocks) {
    using T2 = pair_t<T>;
    using M = Mfma<double>;
    const int kbp = P.sk * P.kc, tid = threadIdx.x, ncb = adj_col_blocks(P);
    const int total = adj_pack_blocks(P, section);
    if (section == 0) {
        // Z[k'][q] = sum over l (in order) of sum_i U[k'-e_l, i] gS_l[i,q] / sigma_q for
        // the l with k' - e_l in I_n; rows padded to whole tiles and columns to cp with zeros
        const int lane = tid & 63, g = lane >> 4, col = lane & 15;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int E = P.n + 2, Pn = P.n + 1, units = P.rt * (P.rows / 16) * ncb, KM = (P.m + 3) >> 2;
        for (int b = block; b < total; b += nblocks) {
            const int unit = kWaves * b + wave;
            if (unit >= units) break;
            const int tile = unit / ncb, q = 16 * (unit - tile * ncb) + col, kr = 16 * tile + col;
            int dig[3] = {0, 0, 0}, rem = kr, idx = 0;
#pragma unroll
            for (int l = 2; l >= 0; --l)
                if (l < P.d) {
                    dig[l] = rem % E;
                    rem /= E;
                }
#pragma unroll
            for (int l = 0; l < 3; ++l)
                if (l < P.d) idx = idx * Pn + dig[l];
            double zr[4] = {0.0, 0.0, 0.0, 0.0}, zi[4] = {0.0, 0.0, 0.0, 0.0};
            int weight = 1;
            for (int l = 1; l < P.d; ++l) weight *= Pn;
#pragma unroll
            for (int ell = 0; ell < 3; ++ell, weight /= Pn) {
                if (ell >= P.d) break;
                bool inside = kr < P.NR && dig[ell] >= 1;
#pragma unroll
                for (int l = 0; l < 3; ++l) inside = inside && (l >= P.d || l == ell || dig[l] <= P.n);
                const double2* u0 = U + (int64_t)(idx - weight) * u_rs;
                const double2* g0 = gS + (size_t)ell * P.m * P.m + q;
                M::acc_t re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
                for (int s = 0; s < KM; s += 4) {
                    double2 u[4], c[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = 4 * (s + k) + g;
                        u[k] = c[k] = make_double2(0.0, 0.0);
                        if (inside && i < P.m) u[k] = u0[i * u_cs];
                        if (q < P.m && i < P.m) c[k] = g0[(size_t)i * P.m];
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (s + k >= KM) break;
                        re = M::fma(u[k].x, c[k].x, re);
                        im = M::fma(u[k].x, c[k].y, im);
                        re = M::fma(-u[k].y, c[k].y, re);
                        im = M::fma(u[k].y, c[k].x, im);
                    }
                }
                // bit r: row r of the tile holds a term of this l
                const unsigned rows = (unsigned)__ballot(inside);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (rows >> M::row(g, r) & 1) {
                        zr[r] += re[r];
                        zi[r] += im[r];
                    }
            }
            if (q < P.cp) {
                const double s = q < P.m ? sigma[q] : 1.0;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    zp[(size_t)(16 * tile + M::row(g, r)) * P.cp + q] = T2{(T)(zr[r] / s), (T)(zi[r] / s)};
            }
        }
    } else if (section == 1) {
        // W = conj(V) as (Re, Im) pairs, row q, column h
        const int tiles = (kbp + 15) / 16 * ncb;
        for (int b = block; b < total; b += nblocks) {
            double2 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = 4 * b + k, hx = 16 * (t / ncb) + (tid & 15), q = 16 * (t % ncb) + (tid >> 4);
                v[k] = make_double2(0.0, 0.0);
                if (hx < P.kb && q < P.m) v[k] = V[hx * v_rs + q * v_cs];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int t = 4 * b + k, hx = 16 * (t / ncb) + (tid & 15), q = 16 * (t % ncb) + (tid >> 4);
                // conj; 0 - 0 keeps the padding +0
                if (t < tiles && hx < kbp && q < P.cp) wp[(size_t)q * kbp + hx] = T2{(T)v[k].x, (T)(0.0 - v[k].y)};
            }
        }
    } else {
        for (int b = block; b < total; b += nblocks)
            for (int x = b * kAdjSpan + tid; x < (b + 1) * kAdjSpan; x += kThreads) {
                if (x < kbp) gt[x] = grid_offset_of_index(x < P.kb ? x : P.kb - 1, P.d, P.n);
                if (x < P.gsize) gf[x] = make_double2(0.0, 0.0);
            }
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void adjoint_pack(AdjPlan P, const double2* __restrict__ U, int64_t u_rs,
                                                    int64_t u_cs, const double* __restrict__ sigma,
                                                    const double2* __restrict__ V, int64_t v_rs, int64_t v_cs,
                                                    const double2* __restrict__ gS, pair_t<T>* __restrict__ zp,
                                                    pair_t<T>* __restrict__ wp, int* __restrict__ gt,
                                                    double2* __restrict__ gf) {
    adj_pack_body<T>(P, U, u_rs, u_cs, sigma, V, v_rs, v_cs, gS, zp, wp, gt, gf, blockIdx.y, blockIdx.x,
                     gridDim.x);
}

// Two 16-row fragments per wave where the rows of Z kept in registers allow it.
constexpr bool adj_rf2_supported(size_t tsize, int ks) { return ks <= (tsize == 4 ? 16 : 8); }

template <typename T>
struct AdjPtrs {
    const pair_t<T>* zp;
    const pair_t<T>* wp;
    const int* gtab;
    double2* gf;
};

// LDS: diagonal bins (2 win_cap doubles: LDS FP64 atomics measured several
// times faster than FP32 ones here, and the bins then add in FP64 for both
// precisions) | h' offsets (kc ints) | two staging
// buffers of one W block (cp rows x 16 pairs each).
__host__ __device__ inline size_t adj_bins_bytes(int win_cap) { return align_up(2 * sizeof(double) * (size_t)win_cap, 16); }
__host__ __device__ inline size_t adj_gt_bytes(int kc) { return align_up(4 * (size_t)kc, 16); }

template <typename T, int KS, int RF>
__device__ __forceinline__ void adjoint_body(const AdjPlan& P, const AdjPtrs<T>& ptr, const int L) {
    using T2 = pair_t<T>;
    using M = Mfma<T>;
    using acc_t = typename M::acc_t;
    constexpr int kTileRows = kRows * RF;
    constexpr int cp = 4 * KS;              // padded complex K
    constexpr int kPairs = cp * kHBlock;          // W pairs of one h block
    constexpr int kBuf = kPairs + 1;              // staging buffer stride: the block and one spare slot
    constexpr int kStg = (kPairs + kThreads - 1) / kThreads;   // staged pairs per thread and block
    extern __shared__ __align__(16) unsigned char smem[];
    double* bins = reinterpret_cast<double*>(smem);      // Re of the window, then Im
    int* gt = reinterpret_cast<int*>(smem + adj_bins_bytes(P.win_cap));
    T2* wst = reinterpret_cast<T2*>(smem + adj_bins_bytes(P.win_cap) + adj_gt_bytes(P.kc));

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, col = lane & 15;
    const int sk_i = L / P.rt, rt_i = L - (L / P.rt) * P.rt;
    const int k_first = rt_i * kTileRows;
    const int k_last = min(k_first + kTileRows - 1, P.NR - 1);
    const int h_first = sk_i * P.kc;
    const int h_last = min(h_first + P.kc, P.kb) - 1;
    const int lo = rowext_offset(k_first, P.d, P.n) - grid_offset_of_index(h_last, P.d, P.n) + P.c0;
    const int hi = rowext_offset(k_last, P.d, P.n) - grid_offset_of_index(h_first, P.d, P.n) + P.c0;
    const int W = hi - lo + 1;
    const int rowlen = P.sk * P.kc;
    const int nblk = P.kc / kHBlock;

    // W block hb: rows q < cp, 16 pairs from column h_first + 16 hb; thread tid
    // moves pairs e = tid + 256 u < cp 16 (row e / 16, pair e % 16). When the
    // block is not a whole number of rounds, the last round's other threads load
    // the block's last pair again (the loads stay unconditional, so the staging
    // registers stay registers) and write nothing.
    auto wsrc = [&](int u, int blk) {
        const int e = min(tid + u * kThreads, kPairs - 1);
        return ptr.wp + (size_t)(e >> 4) * rowlen + (e & 15) + h_first + kHBlock * blk;
    };
    constexpr int kTail = kPairs % kThreads;
    const bool tail_ok = kTail == 0 || tid < kTail;
    // LDS slot of staged pair u: its place in the block, or the buffer's spare slot
    // for the last round's idle threads (every thread writes: no branch)
    auto slot = [&](int u) { return u + 1 < kStg || tail_ok ? tid + u * kThreads : kPairs; };
    static_assert(kStg <= 2, "m <= 32: at most two staged pairs per thread");
    // two named registers rather than an array, which the compiler kept in scratch
    T2 stg0 = *wsrc(0, 0), stg1{};
    if constexpr (kStg > 1) stg1 = *wsrc(1, 0);
    for (int i = tid; i < W; i += kThreads) bins[i] = bins[P.win_cap + i] = 0.0;
    for (int i = tid; i < P.kc; i += kThreads) gt[i] = ptr.gtab[min(h_first + i, h_last)];

    // Element r of lane group g of fragment f is row 4 RF g + 4 f + r of the wave's rows: the
    // lanes of one atomic add then meet in a bin (rows and columns one apart share their
    // diagonal) at most 4 / RF at a time.
    const int krow0 = k_first + 16 * RF * wave;
    auto row_of = [](int f, int grp, int r) { return 4 * RF * grp + 4 * f + r; };
    // A operand (rows of Z) for all K steps, kept in registers
    T2 a[RF][KS];
#pragma unroll
    for (int f = 0; f < RF; ++f)
#pragma unroll
        for (int s = 0; s < KS; ++s)
            a[f][s] = ptr.zp[(size_t)(krow0 + row_of(f, M::group_of_row(col), M::elem_of_row(col))) * cp + 4 * s + g];
    // diagonal bin base of the rows this lane's accumulator elements hold
    int gk[RF][4];
#pragma unroll
    for (int f = 0; f < RF; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            gk[f][r] = rowext_offset(min(krow0 + row_of(f, g, r), P.NR - 1), P.d, P.n) + P.c0 - lo;
    wst[slot(0)] = stg0;
    if constexpr (kStg > 1) wst[slot(1)] = stg1;
    __syncthreads();

    for (int hb = 0; hb < nblk; ++hb) {
        // next block's W (the last block fetches itself again) lands while the MFMAs run
        const int nxt = min(hb + 1, nblk - 1);
        stg0 = *wsrc(0, nxt);
        if constexpr (kStg > 1) stg1 = *wsrc(1, nxt);
        // three real products per complex product: P1 = Re z Re w, P2 = Im z Im w,
        // P3 = (Re z + Im z)(Re w + Im w); Re = P1 - P2, Im = P3 - P1 - P2
        const T2* wb = wst + (hb & 1) * kBuf + g * kHBlock + col;
        acc_t acc[RF][3];
#pragma unroll
        for (int f = 0; f < RF; ++f) acc[f][0] = acc[f][1] = acc[f][2] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const T2 b = wb[4 * s * kHBlock];
            const T bsum = b.x + b.y;
#pragma unroll
            for (int f = 0; f < RF; ++f) acc[f][0] = M::fma(a[f][s].x, b.x, acc[f][0]);
#pragma unroll
            for (int f = 0; f < RF; ++f) acc[f][1] = M::fma(a[f][s].y, b.y, acc[f][1]);
#pragma unroll
            for (int f = 0; f < RF; ++f) acc[f][2] = M::fma(a[f][s].x + a[f][s].y, bsum, acc[f][2]);
        }
        // element r of lane (g, col) of fragment f: row row_of(f, g, r), column
        // h = 16 hb + col (rows past the last row of Z are zero rows: they add zeros)
        const int gh = gt[hb * kHBlock + col];
#pragma unroll
        for (int f = 0; f < RF; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T p1 = acc[f][0][r], p2 = acc[f][1][r], p3 = acc[f][2][r];
                double* bin = &bins[gk[f][r] - gh];
                atomicAdd(bin, (double)(p1 - p2));
                atomicAdd(bin + P.win_cap, (double)(p3 - p1 - p2));
            }
        // the other buffer was last read before the previous barrier
        wst[((hb + 1) & 1) * kBuf + slot(0)] = stg0;
        if constexpr (kStg > 1) wst[((hb + 1) & 1) * kBuf + slot(1)] = stg1;
        __syncthreads();
    }
    double* out = reinterpret_cast<double*>(ptr.gf + lo);
    for (int i = tid; i < 2 * W; i += kThreads) {
        const double v = bins[i & 1 ? P.win_cap + (i >> 1) : i >> 1];
        if (v != 0.0) unsafeAtomicAdd(&out[i], v);
    }
}

template <typename T, int KS, int RF>
__global__ __launch_bounds__(kThreads) void adjoint_tiles(AdjPlan P, AdjPtrs<T> ptr) {
    const int id = blockIdx.x;
    const int L = (P.nwg & 7) == 0 ? (id & 7) * (P.nwg >> 3) + (id >> 3) : id;
    adjoint_body<T, KS, RF>(P, ptr, L);
}

// ---- the smallest FP64 gradients, d >= 2 -----------------------------------------
//
// For one offset p_o of the outer axes 1..d-1 the gradient's line along the last axis is
//     grad(p_o, p) = sum_{k - h = p} G[k, h],
//     G[k, h] = sum over k_o - h_o = p_o and q of Z[(k_o, k), q] conj(V[(h_o, h), q]),
// with n + 2 <= 16 one 16 x 16 tile whose contraction runs over all pairs of lines at that
// offset and over q, and whose diagonals are summed once: no bins, no atomics, a fixed order.
// The offsets x and x - (n + 1), x = 1..n+1, of an outer axis hold n + 2 pairs of lines
// together: line k meets h = k - x from k = x on, and h = k - x + n + 1 before. So each of
// the (n+1)^(d-1) tuples of x has (n+2)^(d-1) pairs in 2^(d-1) runs of one offset, dealt out
// over a workgroup's waves.
//   Two launches (Z, this) instead of the line-spectral form's three: d=2 n=7 m=8 12.2 us
// against 15.8 (the tiles: 12.5), d=3 n=3 m=11 15.0 against 16.9; by 150 pairs times K steps
// the two meet (d=3 n=5 m=11 17.5 against 17.3; at d=3 n=15 m=20 118 against 35), see small_lines.
constexpr int kLineWaves = 8, kLineThreads = 64 * kLineWaves, kLinePairs = 128;

bool small_lines(int d, int n, int m) {
    return d >= 2 && n + 2 <= 16 && ipow(n + 2, d - 1) * ((m + 3) / 4) <= kLinePairs;
}
size_t lines_lds(int d, int n) { return sizeof(double2) * kLineWaves * (16 * 17 + ((size_t)(2 * n + 2) << (d - 1))); }

// A run of pairs of lines at one offset: sides s1, s2 of the outer axes (d = 2: the first is
// trivial), the next pair (i1, i2) of its n1 x n2 pairs, how many are left; the rows of Z and
// of V where the lines of a pair start.
struct LineRun {
    int s1, s2, i1, i2, n2, left;
};
struct LineAxes {
    int d, n, x1, x2;
    __device__ __forceinline__ int n1(int s) const { return d == 2 ? s : s ? n + 2 - x1 : x1; }
    __device__ __forceinline__ int n2(int s) const { return s ? n + 2 - x2 : x2; }
    __device__ __forceinline__ LineRun at(int idx) const {
        int q = d == 2 ? 2 : 0;
        while (idx >= n1(q >> 1) * n2(q & 1)) idx -= n1(q >> 1) * n2(q & 1), ++q;
        const int len = n2(q & 1);
        return LineRun{q >> 1, q & 1, idx / len, idx % len, len, n1(q >> 1) * len - idx};
    }
    __device__ __forceinline__ int z_row(const LineRun& r, int i1, int i2) const {
        const int l1 = r.s1 && d == 3 ? x1 + i1 : i1, l2 = r.s2 ? x2 + i2 : i2;
        return (l1 * (n + 2) + l2) * (n + 2);
    }
    __device__ __forceinline__ int v_row(const LineRun& r, int i1, int i2) const {
        const int h1 = r.s1 ? i1 : i1 + n + 1 - x1, h2 = r.s2 ? i2 : i2 + n + 1 - x2;
        return (h1 * (n + 1) + h2) * (n + 1);
    }
};

// One point from its own terms (where a zero row of Z, of a k' that no T_l holds, met an
// entry that is not finite).
__device__ double2 line_point(const AdjPlan& P, const double2* __restrict__ Z, const double2* __restrict__ V,
                              int64_t v_rs, int64_t v_cs, const int (&p)[3]) {
    const int n = P.n, E = n + 1, a0 = P.d == 3 ? 0 : 1;       // axes a0 .. 2 are the gradient's
    double2 sum = make_double2(0.0, 0.0);
    for (int h = 0; h < P.N; ++h) {
        int rest = h, row = 0, top = 0, zero = 1, k[3] = {0, 0, 0};
        for (int a = 2; a >= a0; --a, rest /= E) k[a] = rest % E + p[a];
        bool inside = true;
        for (int a = a0; a < 3; ++a) {
            inside = inside && k[a] >= 0 && k[a] <= E;
            row = row * (n + 2) + k[a];
            top += k[a] == E;
            zero &= k[a] == 0;
        }
        if (!inside || top > 1 || zero) continue;
        for (int q = 0; q < P.m; ++q) {
            const double2 z = Z[(int64_t)row * P.cp + q], v = V[h * v_rs + q * v_cs];
            sum.x = fma(z.x, v.x, fma(z.y, v.y, sum.x));
            sum.y = fma(z.y, v.x, fma(-z.x, v.y, sum.y));
        }
    }
    return sum;
}

__global__ __launch_bounds__(kLineThreads) void adjoint_lines(AdjPlan P, const double2* __restrict__ Z,
                                                              const double2* __restrict__ V, int64_t v_rs,
                                                              int64_t v_cs, double2* __restrict__ gf) {
    using M = Mfma<double>;
    constexpr int CH = 4;                // K steps in flight
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = P.n, E = n + 1, L = 2 * E, KM = (P.m + 3) >> 2, chunks = (KM + CH - 1) / CH;
    const int len = L << (P.d - 1), lines = P.d == 3 ? (n + 2) * (n + 2) : n + 2, pair = blockIdx.x;
    double2* tile = reinterpret_cast<double2*>(smem) + wave * 16 * 17;
    double2* const all = reinterpret_cast<double2*>(smem) + kLineWaves * 16 * 17;      // [wave][run][place]
    double2* sums = all + (size_t)wave * len;
    // (the hardware keeps a wave's LDS accesses in order; this is for the compiler)
    auto wave_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int i = lane; i < len; i += 64) sums[i] = make_double2(0.0, 0.0);
    const LineAxes X{P.d, n, 1 + pair / E, 1 + pair % E};
    // rows and columns past the last read the last one again: left out below
    const double2* za = Z + (int64_t)min(col, E) * P.cp + g;
    const double2* va = V + (int64_t)min(col, n) * v_rs;
    const int end = lines * (wave + 1) / kLineWaves;
    for (int it = lines * wave / kLineWaves; it < end;) {
        const LineRun run = X.at(it);
        const int count = min(end - it, run.left), steps = count * chunks;
        typename M::acc_t re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
        int i1 = run.i1, i2 = run.i2, c = 0, now = 0;      // step to load next, chunk to multiply next
        auto load = [&](double2 (&z)[CH], double2 (&v)[CH]) {
            const double2* zl = za + (int64_t)X.z_row(run, i1, i2) * P.cp;
            const double2* vl = va + (int64_t)X.v_row(run, i1, i2) * v_rs;
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int s = c * CH + k;
                if (s >= KM) break;
                z[k] = zl[4 * s];
                v[k] = vl[(int64_t)min(4 * s + g, P.m - 1) * v_cs];      // Z is zero past m
            }
            if (++c == chunks) {
                c = 0;
                if (++i2 == run.n2) i2 = 0, ++i1;
            }
        };
        auto mma = [&](const double2 (&z)[CH], const double2 (&v)[CH]) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                if (now * CH + k >= KM) break;
                re = M::fma(z[k].x, v[k].x, re);
                im = M::fma(z[k].y, v[k].x, im);
                re = M::fma(z[k].y, v[k].y, re);
                im = M::fma(-z[k].x, v[k].y, im);
            }
            now = now + 1 == chunks ? 0 : now + 1;
        };
        double2 z0[CH], z1[CH], v0[CH], v1[CH];
        load(z0, v0);
        for (int s = 0; s < steps; s += 2) {
            if (s + 1 < steps) load(z1, v1);
            mma(z0, v0);
            if (s + 1 >= steps) break;
            if (s + 2 < steps) load(z0, v0);
            mma(z1, v1);
        }
        wave_order();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = M::row(g, r);
            tile[col * 17 + row] = row <= E && col <= n ? make_double2(re[r], im[r]) : make_double2(0.0, 0.0);
        }
        wave_order();
        // lane 2 e + comp sums the diagonal k - h = e - 15
        const int e = lane >> 1, place = e - 15 + n;
        if (e < 31 && place >= 0 && place < L) {
            const double* y = reinterpret_cast<const double*>(tile) + (lane & 1);
            const int h0 = max(0, 15 - e), h1 = min(15, 30 - e);
            double sum = 0.0;
#pragma unroll
            for (int h = 0; h < 16; ++h) {
                const int hc = min(max(h, h0), h1);
                const double a = y[2 * (hc * 17 + e - 15 + hc)];
                sum += h >= h0 && h <= h1 ? a : 0.0;
            }
            const int quad = P.d == 2 ? run.s2 : 2 * run.s1 + run.s2;
            reinterpret_cast<double*>(sums + quad * L + place)[lane & 1] += sum;
        }
        it += count;
    }
    __syncthreads();
    for (int e = tid; e < len; e += kLineThreads) {
        double2 v = all[e];
#pragma unroll
        for (int w = 1; w < kLineWaves; ++w) {
            v.x += all[(size_t)w * len + e].x;
            v.y += all[(size_t)w * len + e].y;
        }
        const int quad = e / L, p2 = quad & 1 ? X.x2 : X.x2 - E, p1 = quad & 2 ? X.x1 : X.x1 - E;
        const int p[3] = {p1, p2, e % L - n};
        if (__builtin_expect(!(fabs(v.x) + fabs(v.y) <= 1.7976931348623157e308), 0))
            v = line_point(P, Z, V, v_rs, v_cs, p);
        gf[((P.d == 3 ? (int64_t)(p1 + n) * L : 0) + p2 + n) * L + e % L] = v;
    }
}

// One instance of a batched adjoint: its plan, packed operands, inputs and the
// offsets of its gS / gf blocks in the caller's concatenated buffers.
template <typename T>
struct AdjEntry {
    AdjPlan P;
    AdjPtrs<T> ptr;        // gf unused (taken from gf_all + gf_off)
    const double2* U;
    const double2* V;
    const double* sigma;
    int64_t gs_off, gf_off;   // complex elements
    int tile_begin;           // first tile of this instance in tile_map
};

template <typename T>
__global__ __launch_bounds__(kThreads) void adjoint_pack_batched(const AdjEntry<T>* __restrict__ entries,
                                                            const BatchSlice* __restrict__ slices,
                                                            const double2* __restrict__ gS_all,
                                                            double2* __restrict__ gf_all) {
    const BatchSlice x = slices[blockIdx.x];
    const AdjEntry<T>& e = entries[x.entry];
    const int m = e.P.m;
    adj_pack_body<T>(e.P, e.U, m, 1, e.sigma, e.V, m, 1, gS_all + e.gs_off, const_cast<pair_t<T>*>(e.ptr.zp),
                     const_cast<pair_t<T>*>(e.ptr.wp), const_cast<int*>(e.ptr.gtab), gf_all + e.gf_off, x.section,
                     x.block, 1 << 30);
}

template <typename T, int KS, int RF>
__global__ __launch_bounds__(kThreads) void adjoint_tiles_batched(const AdjEntry<T>* __restrict__ entries,
                                                                  const int* __restrict__ map, int first,
                                                                  double2* __restrict__ gf_all) {
    const int id = first + blockIdx.x;
    const AdjEntry<T>& e = entries[map[id]];
    AdjPtrs<T> ptr = e.ptr;
    ptr.gf = gf_all + e.gf_off;
    adjoint_body<T, KS, RF>(e.P, ptr, id - e.tile_begin);
}

// A single adjoint aims at two workgroups per CU; a batch member splits its h
// range only into chunks of about 256 (long enough to amortise the window flush;
// the batch fills the GPU).
prony_status_t make_adj_plan(prony_handle_t h, int d, int n, int m, size_t tsize, AdjPlan& P, bool batched = false) {
    P = AdjPlan{};
    P.d = d;
    P.n = n;
    P.N = (int)ipow(n + 1, d);
    P.m = m;
    P.NR = (int)ipow(n + 2, d);
    P.cp = (int)align_up((size_t)m, 8);
    P.ksteps = P.cp / 4;
    P.kb = P.N;
    P.rf = adj_rf2_supported(tsize, P.ksteps) && P.NR > kRows ? 2 : 1;
    P.rows = kRows * P.rf;
    P.rt = (P.NR + P.rows - 1) / P.rows;
    P.c0 = grid_center(d, n);
    P.gsize = (int)ipow(2 * n + 2, d);
    const size_t staging = 2 * (2 * tsize) * ((size_t)P.cp * kHBlock + 1);
    const size_t budget = std::min<size_t>(h->lds_per_block, staging + 64 * 1024);
    const int target = batched ? P.rt * std::max(1, P.kb / 256) : 2 * h->num_cus;
    const int sk_target = std::max(1, target / P.rt);
    int kc = (int)align_up((size_t)((P.kb + sk_target - 1) / sk_target), kHBlock);
    kc = std::max(kc, std::min(128, (int)align_up((size_t)P.kb, kHBlock)));
    auto span = [&](int count, int len, bool rowext) {
        int best = 0;
        for (int s = 0; s < count; s += len) {
            const int e = std::min(s + len, count) - 1;
            const int a = rowext ? rowext_offset(s, d, n) : grid_offset_of_index(s, d, n);
            const int b = rowext ? rowext_offset(e, d, n) : grid_offset_of_index(e, d, n);
            best = std::max(best, b - a);
        }
        return best;
    };
    const int rowspan = span(P.NR, P.rows, true);
    for (;;) {
        const int win = rowspan + span(P.kb, kc, false) + 1;
        const size_t lds = adj_bins_bytes(win) + adj_gt_bytes(kc) + staging;
        if (lds <= budget) {
            P.kc = kc;
            P.sk = (P.kb + kc - 1) / kc;
            P.win_cap = win;
            P.lds_bytes = lds;
            break;
        }
        if (kc <= kHBlock) return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint: window does not fit in LDS");
        kc = (int)align_up((size_t)(kc / 2), kHBlock);
    }
    P.nwg = P.rt * P.sk;
    const size_t t2 = 2 * tsize;
    if ((int64_t)P.cp * P.sk * P.kc >= (int64_t(1) << 31))
        return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint: problem too large");
    size_t off = 0;
    P.off_z = off;
    off = align_up(off + t2 * (size_t)P.rt * P.rows * P.cp, 256);
    P.off_w = off;
    off = align_up(off + t2 * (size_t)P.cp * P.sk * P.kc, 256);
    P.off_g = off;
    off = align_up(off + 4 * (size_t)P.sk * P.kc, 256);
    P.ws_bytes = off;
    return PRONY_OK;
}

template <typename T, int KS, int RF>
prony_status_t launch_adj_tiles(prony_handle_t h, const AdjPlan& P, const AdjPtrs<T>& ptr) {
    if (P.lds_bytes > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&adjoint_tiles<T, KS, RF>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)P.lds_bytes);
        if (e != hipSuccess) return hip_fail(h, e, "hipFuncSetAttribute");
    }
    ProfileScope prof(h, "adjoint_tiles");
    adjoint_tiles<T, KS, RF><<<P.nwg, kThreads, P.lds_bytes, h->stream>>>(P, ptr);
    return PRONY_OK;
}

template <typename T, int KS>
prony_status_t dispatch_adj_tiles(prony_handle_t h, const AdjPlan& P, const AdjPtrs<T>& ptr) {
    if constexpr (adj_rf2_supported(sizeof(T), KS))
        if (P.rf == 2) return launch_adj_tiles<T, KS, 2>(h, P, ptr);
    return launch_adj_tiles<T, KS, 1>(h, P, ptr);
}

template <typename T>
prony_status_t launch_adjoint(prony_handle_t h, const AdjPlan& P, const double* U, int64_t u_rs, int64_t u_cs,
                              const double* sigma, const double* V, int64_t v_rs, int64_t v_cs, const double* gS,
                              double* gf) {
    using T2 = pair_t<T>;
    prony_status_t st = ensure_workspace(h, P.ws_bytes);
    if (st != PRONY_OK) return st;
    unsigned char* ws = static_cast<unsigned char*>(h->ws);
    T2* zp = reinterpret_cast<T2*>(ws + P.off_z);
    T2* wp = reinterpret_cast<T2*>(ws + P.off_w);
    int* gt = reinterpret_cast<int*>(ws + P.off_g);
    const int blocks = std::min(std::max({adj_pack_blocks(P, 0), adj_pack_blocks(P, 1), adj_pack_blocks(P, 2)}),
                                2 * h->num_cus);
    {
        ProfileScope prof(h, "adjoint_pack");
        adjoint_pack<T><<<dim3(blocks, 3), kThreads, 0, h->stream>>>(
            P, reinterpret_cast<const double2*>(U), u_rs, u_cs, sigma, reinterpret_cast<const double2*>(V), v_rs,
            v_cs, reinterpret_cast<const double2*>(gS), zp, wp, gt, reinterpret_cast<double2*>(gf));
    }
    if ((st = check_launch(h, "adjoint_pack")) != PRONY_OK) return st;
    const AdjPtrs<T> ptr{zp, wp, gt, reinterpret_cast<double2*>(gf)};
    switch (P.ksteps) {
#define PRONY_ADJ_CASE(K) \
    case K:               \
        st = dispatch_adj_tiles<T, K>(h, P, ptr); \
        break;
        PRONY_ADJ_CASE(2)
        PRONY_ADJ_CASE(4)
        PRONY_ADJ_CASE(6)
        PRONY_ADJ_CASE(8)
#undef PRONY_ADJ_CASE
        default:
            return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint: m too large");
    }
    if (st != PRONY_OK) return st;
    return check_launch(h, "adjoint_tiles");
}

// The two launches of one of the smallest gradients; the workspace holds Z.
prony_status_t launch_lines(prony_handle_t h, AdjPlan P, const double* U, int64_t u_rs, int64_t u_cs,
                            const double* sigma, const double* V, int64_t v_rs, int64_t v_cs, const double* gS,
                            double* gf) {
    prony_status_t st = ensure_workspace(h, P.ws_bytes);
    if (st != PRONY_OK) return st;
    double2* Z = reinterpret_cast<double2*>(static_cast<unsigned char*>(h->ws) + P.off_z);
    {
        ProfileScope prof(h, "adjoint_pack");
        adjoint_pack<double><<<dim3(adj_pack_blocks(P, 0), 1), kThreads, 0, h->stream>>>(
            P, reinterpret_cast<const double2*>(U), u_rs, u_cs, sigma, reinterpret_cast<const double2*>(V), v_rs,
            v_cs, reinterpret_cast<const double2*>(gS), Z, nullptr, nullptr, nullptr);
    }
    if ((st = check_launch(h, "adjoint_pack")) != PRONY_OK) return st;
    {
        ProfileScope prof(h, "adjoint_lines");
        adjoint_lines<<<(int)ipow(P.n + 1, P.d - 1), kLineThreads, lines_lds(P.d, P.n), h->stream>>>(
            P, Z, reinterpret_cast<const double2*>(V), v_rs, v_cs, reinterpret_cast<double2*>(gf));
    }
    return check_launch(h, "adjoint_lines");
}

template <typename T, int KS>
prony_status_t launch_adj_batched_ks(prony_handle_t h, int rf, const AdjEntry<T>* entries, const int* map, int first,
                                     int tiles, size_t lds, double2* gf) {
    if constexpr (adj_rf2_supported(sizeof(T), KS))
        if (rf == 2) {
            if (lds > 65536) {
                hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&adjoint_tiles_batched<T, KS, 2>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                if (e != hipSuccess) return hip_fail(h, e, "hipFuncSetAttribute");
            }
            ProfileScope prof(h, "adjoint_tiles_batched");
            adjoint_tiles_batched<T, KS, 2><<<tiles, kThreads, lds, h->stream>>>(entries, map, first, gf);
            return PRONY_OK;
        }
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&adjoint_tiles_batched<T, KS, 1>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return hip_fail(h, e, "hipFuncSetAttribute");
    }
    ProfileScope prof(h, "adjoint_tiles_batched");
    adjoint_tiles_batched<T, KS, 1><<<tiles, kThreads, lds, h->stream>>>(entries, map, first, gf);
    return PRONY_OK;
}

}  // namespace

struct AdjBatch {
    void* ws = nullptr;           // device AdjEntry<T>[count] (grouped by class), then operands
    int count = 0;
    const BatchSlice* slices = nullptr;   // device, a packing workgroup each
    const int* tile_map = nullptr;        // device, the entry of every tile
    int packs = 0;
    int64_t gs_elems = 0, gf_elems = 0;   // complex elements of the concatenated gS / gf
    struct ClassLaunch {
        int ks, rf, first, tiles;         // first tile in tile_map
        size_t lds;
    };
    std::vector<ClassLaunch> launches;
    SpecAdjBatch* spec = nullptr;   // FP64 in line-spectral form: replaces the tiles above
};

prony_status_t adj_batch_free(AdjBatch* a) {
    prony_status_t st = PRONY_OK;
    if (a->ws && hipFree(a->ws) != hipSuccess) st = PRONY_EHIP;
    if (a->spec && spectral_adjoint_batch_free(a->spec) != PRONY_OK) st = PRONY_EHIP;
    delete a;
    return st;
}

namespace {

template <typename T>
prony_status_t adj_batch_build(prony_handle_t h, const prony_batch_s* B, AdjBatch* A) {
    using T2 = pair_t<T>;
    const int count = B->count;
    std::vector<AdjPlan> plans(count);
    std::vector<int64_t> gs_off(count), gf_off(count);
    for (int i = 0; i < count; ++i) {
        const prony_instance_t& x = B->inst[i];
        prony_status_t st = make_adj_plan(h, x.d, x.n, x.m, sizeof(T), plans[i], true);
        if (st != PRONY_OK) return fail(h, st, "instance " + std::to_string(i) + ": " + h->err);
        gs_off[i] = A->gs_elems;
        A->gs_elems += (int64_t)x.d * x.m * x.m;
        gf_off[i] = A->gf_elems;
        A->gf_elems += plans[i].gsize;
    }
    // FP64 in line-spectral form where every instance fits it and its memory can be had
    if (sizeof(T) == 8 && !B->direct) {
        const prony_status_t st = spectral_adjoint_batch_build(h, B->inst, gs_off, gf_off, &A->spec);
        if (st == PRONY_OK || st == PRONY_EHIP) return st;
        h->err.clear();
    }
    // classes by (K steps, fragments); inside a class, most workgroups first
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        if (plans[a].ksteps != plans[b].ksteps) return plans[a].ksteps < plans[b].ksteps;
        if (plans[a].rf != plans[b].rf) return plans[a].rf < plans[b].rf;
        return plans[a].nwg > plans[b].nwg;
    });
    std::vector<BatchSlice> packs;
    for (int pos = 0; pos < count; ++pos)
        for (int section = 0; section < 3; ++section)
            for (int b = 0; b < adj_pack_blocks(plans[order[pos]], section); ++b) packs.push_back({pos, section, b});
    if (packs.size() > (size_t)INT32_MAX / 2)
        return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint_batched: too many instances");
    const size_t off_packs = align_up(sizeof(AdjEntry<T>) * (size_t)count, 256);
    std::vector<int> tile_map;      // class after class
    for (int pos = 0; pos < count; ++pos) tile_map.insert(tile_map.end(), (size_t)plans[order[pos]].nwg, pos);
    if (tile_map.size() > (size_t)INT32_MAX)
        return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint_batched: too many tiles");
    const size_t off_map = align_up(off_packs + sizeof(BatchSlice) * packs.size(), 256);
    size_t off = align_up(off_map + sizeof(int) * tile_map.size(), 256);
    std::vector<size_t> base(count);
    for (int pos = 0; pos < count; ++pos) {
        base[pos] = off;
        off = align_up(off + plans[order[pos]].ws_bytes, 256);
    }
    hipError_t e = hipMalloc(&A->ws, off);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        A->ws = nullptr;
        return fail(h, PRONY_ENOMEM, std::string("batch adjoint workspace allocation failed: ") + hipGetErrorString(e));
    }
    unsigned char* w = static_cast<unsigned char*>(A->ws);
    std::vector<AdjEntry<T>> host(count);
    int first = 0;
    for (int pos = 0; pos < count; ++pos) {
        const int i = order[pos];
        const AdjPlan& P = plans[i];
        const prony_instance_t& x = B->inst[i];
        AdjEntry<T>& E = host[pos];
        E.P = P;
        E.ptr.zp = reinterpret_cast<const T2*>(w + base[pos] + P.off_z);
        E.ptr.wp = reinterpret_cast<const T2*>(w + base[pos] + P.off_w);
        E.ptr.gtab = reinterpret_cast<const int*>(w + base[pos] + P.off_g);
        E.ptr.gf = nullptr;
        E.U = reinterpret_cast<const double2*>(x.U);
        E.V = reinterpret_cast<const double2*>(x.V);
        E.sigma = x.sigma;
        E.gs_off = gs_off[i];
        E.gf_off = gf_off[i];
        const bool new_class = pos == 0 || plans[order[pos - 1]].ksteps != P.ksteps ||
                               plans[order[pos - 1]].rf != P.rf;
        if (new_class) A->launches.push_back({P.ksteps, P.rf, first, 0, 0});
        auto& cl = A->launches.back();
        E.tile_begin = first;
        first += P.nwg;
        cl.tiles = first - cl.first;
        cl.lds = std::max(cl.lds, P.lds_bytes);
    }
    A->count = count;
    A->slices = reinterpret_cast<const BatchSlice*>(w + off_packs);
    A->tile_map = reinterpret_cast<const int*>(w + off_map);
    A->packs = (int)packs.size();
    e = hipMemcpyAsync(A->ws, host.data(), sizeof(AdjEntry<T>) * (size_t)count, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(w + off_packs, packs.data(), sizeof(BatchSlice) * packs.size(), hipMemcpyHostToDevice,
                           h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(w + off_map, tile_map.data(), sizeof(int) * tile_map.size(), hipMemcpyHostToDevice,
                           h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "batch adjoint work table upload");
    return PRONY_OK;
}

template <typename T>
prony_status_t adj_batch_launch(prony_handle_t h, const AdjBatch* A, const double* gS, double* gf) {
    if (A->spec) return spectral_adjoint_batch_launch(h, A->spec, gS, gf);
    const AdjEntry<T>* entries = static_cast<const AdjEntry<T>*>(A->ws);
    const double2* gs2 = reinterpret_cast<const double2*>(gS);
    double2* gf2 = reinterpret_cast<double2*>(gf);
    {
        ProfileScope prof(h, "adjoint_pack");
        adjoint_pack_batched<T><<<A->packs, kThreads, 0, h->stream>>>(entries, A->slices, gs2, gf2);
    }
    prony_status_t st = check_launch(h, "adjoint_pack_batched");
    if (st != PRONY_OK) return st;
    for (const auto& cl : A->launches) {
        switch (cl.ks) {
#define PRONY_ADJ_BCASE(K)                                                                              \
    case K:                                                                                             \
        st = launch_adj_batched_ks<T, K>(h, cl.rf, entries, A->tile_map, cl.first, cl.tiles, cl.lds, gf2);    \
        break;
            PRONY_ADJ_BCASE(2)
            PRONY_ADJ_BCASE(4)
            PRONY_ADJ_BCASE(6)
            PRONY_ADJ_BCASE(8)
#undef PRONY_ADJ_BCASE
            default:
                return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint_batched: m too large");
        }
        if (st != PRONY_OK) return st;
        if ((st = check_launch(h, "adjoint_tiles_batched")) != PRONY_OK) return st;
    }
    return PRONY_OK;
}

}  // namespace

size_t adjoint_workspace_bytes(prony_handle_t h, int d, int n, int m) {
    size_t best = 0;
    for (size_t ts : {sizeof(float), sizeof(double)}) {
        AdjPlan P;
        if (make_adj_plan(h, d, n, m, ts, P) == PRONY_OK) best = std::max(best, P.ws_bytes);
    }
    return best;
}

}  // namespace prony

using namespace prony;

extern "C" prony_status_t prony_build_S_adjoint(prony_handle_t h, int d, int n, int m, const double* U,
                                                int64_t u_rs, int64_t u_cs, const double* sigma, const double* V,
                                                int64_t v_rs, int64_t v_cs, const double* gS, prony_prec_t prec,
                                                double* gf) {
    if (!h) return PRONY_EINVAL;
    prony_status_t st = check_dn(h, d, n);
    if (st != PRONY_OK) return st;
    const int64_t N = ipow(n + 1, d);
    if (m < 1 || m > N) return fail(h, PRONY_EINVAL, "prony_build_S_adjoint: m must be in 1..N");
    if (m > 32) return fail(h, PRONY_ENOTSUP, "prony_build_S_adjoint: m > 32 is not supported");
    if (!U || !V || !sigma || !gS || !gf) return fail(h, PRONY_EINVAL, "prony_build_S_adjoint: null pointer");
    if (u_rs < 1 || u_cs < 1 || v_rs < 1 || v_cs < 1)
        return fail(h, PRONY_EINVAL, "prony_build_S_adjoint: strides must be >= 1");
    if ((N - 1) * u_rs + (m - 1) * u_cs >= (int64_t(1) << 40) || (N - 1) * v_rs + (m - 1) * v_cs >= (int64_t(1) << 40))
        return fail(h, PRONY_EINVAL, "prony_build_S_adjoint: strides out of range");
    if (prec != PRONY_FP64 && prec != PRONY_FP64_DIRECT && prec != PRONY_FP32)
        return fail(h, PRONY_EINVAL, "prony_build_S_adjoint: bad precision");
    if (h->device < 0) return fail(h, PRONY_ENODEV, "validation-only handle has no device");
    DeviceGuard g(h->device);
    if (!g.ok) return fail(h, PRONY_EHIP, "hipSetDevice failed");
    AdjPlan P;
    if (prec == PRONY_FP32) {
        if ((st = make_adj_plan(h, d, n, m, sizeof(float), P)) != PRONY_OK) return st;
        return launch_adjoint<float>(h, P, U, u_rs, u_cs, sigma, V, v_rs, v_cs, gS, gf);
    }
    if ((st = make_adj_plan(h, d, n, m, sizeof(double), P)) != PRONY_OK) return st;
    const bool direct = prec == PRONY_FP64_DIRECT;
    if (!direct && small_lines(d, n, m))
        return launch_lines(h, P, U, u_rs, u_cs, sigma, V, v_rs, v_cs, gS, gf);
    // in line-spectral form where it applies (a shape the tiles cannot cover is refused above)
    SpecPlan SP{};
    bool spectral = !direct && spectral_adjoint_plan(h, d, n, m, SP);
    if ((st = ensure_form(h, SP.ws_bytes, P.ws_bytes, spectral)) != PRONY_OK) return st;
    if (spectral)
        return spectral_adjoint_run(h, SP, static_cast<unsigned char*>(h->ws), U, u_rs, u_cs, sigma, V, v_rs, v_cs,
                                    gS, gf);
    return launch_adjoint<double>(h, P, U, u_rs, u_cs, sigma, V, v_rs, v_cs, gS, gf);
}

extern "C" prony_status_t prony_build_S_adjoint_batched(prony_handle_t h, prony_batch_t B, const double* gS,
                                                        double* gf) {
    if (!h || !B) return PRONY_EINVAL;
    if (B->owner != h) return fail(h, PRONY_EINVAL, "prony_build_S_adjoint_batched: batch belongs to another handle");
    if (!gS || !gf) return fail(h, PRONY_EINVAL, "prony_build_S_adjoint_batched: null pointer");
    if (h->device < 0) return fail(h, PRONY_ENODEV, "validation-only handle has no device");
    DeviceGuard g(h->device);
    if (!g.ok) return fail(h, PRONY_EHIP, "hipSetDevice failed");
    if (!B->adj) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(h->stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
            return fail(h, PRONY_ECAPTURE,
                        "prony_build_S_adjoint_batched: the first call on a batch plans and allocates; "
                        "make it outside stream capture");
        AdjBatch* A = new (std::nothrow) AdjBatch();
        if (!A) return fail(h, PRONY_ENOMEM, "prony_build_S_adjoint_batched: out of host memory");
        const prony_status_t st = B->prec == PRONY_FP32 ? adj_batch_build<float>(h, B, A)
                                                        : adj_batch_build<double>(h, B, A);
        if (st != PRONY_OK) {
            (void)adj_batch_free(A);
            return st;
        }
        B->adj = A;
    }
    return B->prec == PRONY_FP32 ? adj_batch_launch<float>(h, B->adj, gS, gf)
                                 : adj_batch_launch<double>(h, B->adj, gS, gf);
}
