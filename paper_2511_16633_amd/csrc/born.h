// Born contraction kernels (adjoint.hip, forward.hip, hessian.hip): parameters and host
// entry points shared with the inversion driver.
#pragma once
#include "common.h"

namespace rb {

struct AdjParams {
    int m, mp, nb, nf;     // nb = mp / 32 blocks of elements
    int64_t N;
    double cg[RB_MAX_NF];  // 2 omega^2 h^2
    double ch[RB_MAX_NF];  // 2 omega^4 h^4
};

// One problem's backprojection as the contraction kernel sees it, for
// launches that group several problems: its parameters, its tables and
// prepared operands, its per-frequency partial sums, its pixel tiles per
// frequency, its first flat workgroup in the launch and how many workgroups
// split the emitter passes of one pixel tile.
struct AdjItem {
    AdjParams P;
    const void *Gr, *Gi, *Ar, *Ai, *Wt;
    const uint8_t *flags;
    const float *gscale, *ascale;
    double *pg, *ph;
    int ntiles, begin;
    int npg;   // emitter-pass groups per pixel tile, each a workgroup of its own (partials [nf][npg][N])
    // FP32 tables on the FP16 cores: split operands, G scales [nf][N], whether
    // a frequency's A does not fit them [nf], and the list of work items to
    // compute in FP32 (its length, then the items)
    void *split_hi, *split_lo;
    const float *pscale;
    int *bad, *redo;
};
constexpr int kAdjGroupMax = 8;   // problems per grouped launch (kernel-argument size)
struct AdjGroup {
    int n;
    AdjItem item[kAdjGroupMax];
};

// A prepared backprojection (operands and block flags written on the
// stream), ready for its contraction kernel alone or grouped with others.
struct AdjTask {
    AdjItem item;
    rb_dtype dt;
    bool split;   // FP32 tables, gradient by k_adjoint_split
    bool direct;  // 16-bit tables: k_adjoint16_tr with direct loads
    double *grad, *hdiag;
};

struct FwdParams {
    int m, mp, nf, ntl, ntri, nsplit;
    int dmin;              // >= 32: pairs closer than this need not be computed
    int64_t N, kchunk;
    bool sum64;            // FP32: the partials are FP64
    double cg[RB_MAX_NF];  // omega^2 h^2
};

size_t adjoint_workspace_bytes(const rb_geometry *g, int nf, rb_dtype dt);
size_t forward_workspace_bytes(const rb_geometry *g, int nf, rb_dtype dt);

// grad/hdiag += (see rb_born_adjoint_weighted); gscale may be null for 32/64-bit.
rb_status adjoint_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                       rb_dtype dt, const double *freqs, int nf, const double *d_res, const double *w_data,
                       double *grad, double *hdiag, void *ws, size_t ws_bytes, hipStream_t st);
// The same as adjoint_impl in two parts: the operand preparation, then the
// contraction and the frequency sum.  adjoint_run_grouped runs the second
// part of several prepared problems, with one contraction launch per
// contraction type (up to kAdjGroupMax problems each); every problem's result
// is bitwise that of adjoint_impl.  The f64 type is prepared and run alone.
rb_status adjoint_prepare(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                          rb_dtype dt, const double *freqs, int nf, const double *d_res, const double *w_data,
                          double *grad, double *hdiag, void *ws, size_t ws_bytes, hipStream_t st, AdjTask *task);
rb_status adjoint_run(const AdjTask &task, hipStream_t st);
rb_status adjoint_run_grouped(AdjTask *const *tasks, int n, hipStream_t st);
// d_out = J delta, [nf][m][m] complex.  With dmin >= 32 (a caller that
// weights every pair of circular index distance below dmin by zero) those
// pairs are returned as 0, whatever the type, and the 32/16-bit kernels skip
// the tiles and blocks that hold no other pair.
rb_status forward_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                       rb_dtype dt, const double *freqs, int nf, const double *delta, double *d_out, void *ws,
                       size_t ws_bytes, hipStream_t st, int dmin = 0);

// hdiag += Hessian diagonal for band-selection weights with zeroed pairs
// (see rb_born_hessian_banded); zeroed: [nf][zcap] (e, r), nzero: [nf].
rb_status hessian_band_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                            rb_dtype dt, const double *freqs, int nf, int dmin, const int *zeroed,
                            const int *nzero, int zcap, double *hdiag, hipStream_t st);

// Argument checks shared by the contraction entry points.
rb_status check_contraction(const rb_geometry *g, const void *G_re, const void *G_im, const float *scale,
                            rb_dtype dt, const double *freqs, int32_t nf);

}  // namespace rb
