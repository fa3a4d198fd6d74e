// Host interface of the solver vector kernels (blas.hip).  Reductions write their results
// (FP64, already summed over the lattice and multiplied by `scale`) to device memory, so a
// solver iteration needs no host round trip except where it reads a norm to decide.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "internal.h"

namespace dl {

// A batch of nrhs systems sharing one lattice: vector r of an argument is r vectors after its
// base, basis vector j of system r is (j * nrhs + r) vectors after the base, and system r's
// device scalars are r * sstride doubles after a scalar pointer.  Systems with active[r] = 0
// are skipped.  The default is one system.
struct BatchSpec {
    int nrhs = 1;
    const int *active = nullptr;
    int sstride = 0;
};

// device scalar slots (doubles) of a system: work-groups finished (an integer, zero between launches), residual
// norm^2 at S_RED + 4, flags of the step (empty, to be corrected) at S_RED + 6, {1 / gamma, estimate of alpha, its
// correction}, free slots, per iteration gamma_k, alpha_k, the solution's coefficients c_k, |Q_k|^2 and the beta_kj
constexpr int kGcrMax = 64;  // longest cycle
constexpr int S_COUNT = 0, S_RED = 0, S_SC = 8, S_MISC = 16, S_GAM = 64, S_ALP = 192, S_C = 320, S_N2 = 448, S_BETA = 512;
constexpr int kSysScal = 8768;  // device scalar doubles per system: GCR(64) coefficients and 64 free slots

struct Blas {
    dirac_ctx *c = nullptr;
    DevBuf part, scal;  // partial sums, scalars

    void reserve(int64_t nsites_max, int nrhs = 1);
    // out = scale <x, y> (complex, 2 doubles)
    void dot(dirac_prec pr, int nh, const void *x, const void *y, double *out_dev, double scale, hipStream_t s,
             const BatchSpec &bs = BatchSpec());
    // Step k of a GCR cycle (basis vectors Q_0 .. Q_{k-1}, q = A p_k): the scalars beta_k and gamma_k and an estimate of
    // alpha_k, then q <- the new basis vector, rnew = r - alpha q (rnew may be r), |rnew|^2 in S_RED + 4, and
    // S_RED + 6 = 1 when nothing was left of q (then rnew = r, and the cycle should end), else 0; with ctl (one
    // system) the iteration control of the cycle is advanced against `target`.  defer: the correction of alpha is
    // left to the caller, who calls gcr_correct where S_RED + 7 is not 0 (with ctl: ctl[3] = 1, ctl[0] = 0 until then).
    void gcr_dots(dirac_prec pr, int nh, const void *Q, int k, const void *q, const void *r, double scale, hipStream_t s,
                  const BatchSpec &bs = BatchSpec());
    void gcr_step(dirac_prec pr, int nh, const void *Q, int k, void *q, const void *r, void *rnew, double scale,
                  hipStream_t s, const BatchSpec &bs = BatchSpec(), int *ctl = nullptr, double target = 0.0,
                  bool defer = false);
    void gcr_correct(dirac_prec pr, int nh, const void *q, void *rnew, double scale, hipStream_t s,
                     const BatchSpec &bs = BatchSpec(), int *ctl = nullptr, double target = 0.0);
    // the coefficients S_C of x += sum_j c_j p_j after a cycle of n steps (counts[sys] when given), zero up to kmax
    void gcr_backsub(const int *counts, int n, int kmax, hipStream_t s, const BatchSpec &bs = BatchSpec());
    // x += xscale sum_j coef_j P_j, j < k (xscale_r = xscales[r * sstride] when given; system r sums
    // only j < kcount[r] when kcount is given)
    void axpy_multi(dirac_prec px, dirac_prec pp, int nh, void *x, const void *P, int k, const double *coef_dev,
                    double xscale, hipStream_t s, const BatchSpec &bs = BatchSpec(), const double *xscales = nullptr,
                    const int *kcount = nullptr);
    // out = alpha a + beta b; copy2 = out; out_dev = scale {|out|^2, nonfinite flag}
    void lincomb(dirac_prec po, dirac_prec pa, dirac_prec pb, int nh, void *out, void *copy2, double alpha,
                 const void *a, double beta, const void *b, double *out_dev, double scale, hipStream_t s,
                 const BatchSpec &bs = BatchSpec(), const double *alphas = nullptr);
    void cgls_xs(int nh, const double *rho, const double *wn, void *x, const void *p, void *sv, const void *w,
                 double *out_dev, hipStream_t s);
    void cgls_p(int nh, const double *rho_new, const double *rho_old, void *p, const void *r, hipStream_t s);
    void set(double *p, double v, hipStream_t s);
    void copy_scalar(const double *src, double *dst, hipStream_t s);
};

int blas_grid(int64_t nsites);

// Solver work space of a context (solver.hip)
struct SolverWork {
    Blas blas;
    DevBuf P, Q, r, e, b;   // Krylov vectors, inner solution / right-hand side (solve precision)
    DevBuf h64[4];          // FP64 half vectors: eta-hat, x_e, r, tmp
    DevBuf ctl;             // device-side iteration control of a GCR cycle (solver.hip)
    DevBuf f64[3];          // FP64 full vectors: b, x, r
    int m = 0;
    dirac_prec pr = DIRAC_F64;
    double *pin = nullptr;  // pinned host memory for the values a solve waits for (8 doubles)
    long syncs = 0;  // host waits on the device (value reads) since the current solve began
    bool correct = false;  // a step of the current solve needed its correction: it follows every step
};

}  // namespace dl
