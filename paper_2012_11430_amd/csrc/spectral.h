// Line-spectral form of the FP64 S-build (spectral.hip): plan, operands, launches.
#pragma once

#include "common.h"

namespace prony {

// Plan of one instance in the line-spectral form. One axis of I_n stays direct
// (K1 lines), the others are transformed on L = 2P points each:
//   d >= 2: axis 1 is direct (K1 = n + 1 lines), axes 2..d have P = n + 1 points;
//   d = 1:  the index k = k1 P + k2 is folded into K1 lines of P points.
struct SpecPlan {
    int d, n, N, m;
    int P, L, K1;
    int pmax;       // largest sample index used: n + 1, products with T: n
    int NP1;        // sample lines p1 = t - (K1 - 1), t < NP1
    int F;          // frequencies: L^(transformed axes)
    int ells, s0;   // stored matrices (S_0 first with s0), d or d + 1
    int npb;        // blocks of 16 frequency pairs along one axis
    // forward transforms
    int nbw;        // d <= 2: 8-column blocks per workgroup (factors)
    int nbwf;       //         the same for the sample lines
    int nq;         // d = 3: factor columns per workgroup (at most 8)
    int splits;     // d = 3: blocks of 16 frequency pairs of axis 3
    int wgs_x;      // workgroups per factor (U, V)
    int wgs_f;      // workgroups of the sample grid
    size_t lds_fwd;
    // weighted Gram products
    int nqb;        // 16-column blocks of V
    int nmb, nm0;   // 16-row blocks of [U | shifted U], those with unshifted rows
    int ns;         // sums kept: 1 with the last axis' phase, 2 plain and with that phase
    int groups;     // groups of frequencies = rows of partials
    int gparts;     // groups per frequency of axis 2 (d = 3), else all groups
    size_t lds_gram;
    // inverse transforms of the products
    int nbi;            // d <= 2: 8-column blocks per workgroup
    int nqi;            // d = 3: columns per workgroup
    int isplits, irows; // d = 3: parts of the folded rows of axis 2, rows per part
    int wgs_i;
    size_t lds_inv;
    // workspace sections (bytes): U~ | V~ | f~ | partials | tables; the first off_f bytes are
    // what prepared factors keep
    size_t off_v, off_f, off_p, off_r, ws_bytes;
};

// Operands of one instance.
struct SpecPtrs {
    const double2* U;
    const double2* V;
    int64_t u_rs, u_cs, v_rs, v_cs;
    const double2* f;
    const double* sigma;
    double2* ut;      // U~[w][k1][i]
    double2* vt;      // V~[w][h1][q]
    double2* ft;      // f~[w][t], scaled by 1/F
    double2* part;    // [group][i][l][q]
    double2* S;
    double2* tables;  // workspace section for the tables where the handle holds none
    const double2* tab;
};

// Plan of an FP64 S-build; false where the form does not apply (see there).
bool spectral_plan(prony_handle_t h, int d, int n, int m, bool s0, SpecPlan& P, bool batched = false);

// Launches on the handle's stream: the transforms of U and V, and/or of the sample
// grid; then the weighted Gram products and the finishing sums into S.
// (sets ptr.tab: the handle's tables, made and kept there on the first use of a line length
// when keep_tables, else made in ptr.tables).
prony_status_t spectral_forward(prony_handle_t h, const SpecPlan& P, SpecPtrs& ptr, bool factors, bool grid,
                                bool keep_tables);
prony_status_t spectral_gram_finish(prony_handle_t h, const SpecPlan& P, const SpecPtrs& ptr);

// Bytes of the tables of a plan; the tables of every shape up to (d_max, n_max), so that
// later calls allocate none.
size_t spectral_table_bytes(const SpecPlan& P);
prony_status_t spectral_reserve(prony_handle_t h, int d_max, int n_max);

// Largest workspace of a single S-build or adjoint of dimension d within the bounds. It
// does not grow with n and m: the groups of frequencies (rows of partials) halve where a
// second column block starts and step with n, and a larger shape may leave the form.
size_t spectral_reserve_bytes(prony_handle_t h, int d, int n_max, int m_max);

// FP64 batches: the plan of all instances with its own device memory (PRONY_ENOTSUP when
// one of them does not fit the form, PRONY_ENOMEM), its launches, its release.
prony_status_t spectral_batch_build(prony_handle_t h, const std::vector<prony_instance_t>& inst, SpecBatch** out);
prony_status_t spectral_batch_launch(prony_handle_t h, const SpecBatch* S);

// Plan of an FP64 product with T or T^* and r columns (the workspace: Y~ | X~ | f~ | tables),
// and the product.
bool spectral_product_plan(prony_handle_t h, int d, int n, int r, SpecPlan& P);
prony_status_t spectral_product(prony_handle_t h, const SpecPlan& P, unsigned char* ws, const double* f,
                                const double* X, int64_t ldx, bool adjoint, double* Y, int64_t ldy);

// Plan of an FP64 adjoint (d >= 2; the workspace: U~ | V~ | g~ | tables), and the adjoint.
bool spectral_adjoint_plan(prony_handle_t h, int d, int n, int m, SpecPlan& P, bool batched = false);
prony_status_t spectral_adjoint_run(prony_handle_t h, const SpecPlan& P, unsigned char* ws, const double* U,
                                    int64_t u_rs, int64_t u_cs, const double* sigma, const double* V, int64_t v_rs,
                                    int64_t v_cs, const double* gS, double* gf);

// FP64 adjoints of a batch (every instance with d >= 2; else as spectral_batch_build).
struct SpecAdjBatch;
prony_status_t spectral_adjoint_batch_build(prony_handle_t h, const std::vector<prony_instance_t>& inst,
                                            const std::vector<int64_t>& gs_off, const std::vector<int64_t>& gf_off,
                                            SpecAdjBatch** out);
prony_status_t spectral_adjoint_batch_launch(prony_handle_t h, const SpecAdjBatch* S, const double* gS, double* gf);
prony_status_t spectral_adjoint_batch_free(SpecAdjBatch* b);

}  // namespace prony
