// Vector kernels of the Krylov solvers on NATIVE vectors (one thread per site, 24 reals).
// Every reduction accumulates in FP64 and is deterministic: each work-group reduces its sites
// in a fixed tree and writes one partial; a second kernel sums the partials in index order.
// No floating-point atomics anywhere.
//
// A "vector" here is nh consecutive half-lattice blocks (nh = 1 for an even-odd vector, 2 for
// a full-lattice vector): block h starts h * 24 vh reals after the base and holds 24 / W planes
// of vh sites.
#include "blas.h"

#include <algorithm>

namespace dl {
namespace {

constexpr int kRed = 256;  // work-group size of the reducing kernels

// (half h, base) of site t of an nh-half vector; halves are 24 / W planes of vhp sites apart
template <typename S>
DEV const typename St<S>::vec *blk_base(const typename St<S>::vec *p, int t, int vh, uint32_t &i) {
    const int h = t >= vh;
    i = (uint32_t)(t - h * vh);
    return p + (size_t)h * (24 / St<S>::W) * (size_t)padded_sites(vh);
}
template <typename S>
DEV typename St<S>::vec *blk_base(typename St<S>::vec *p, int t, int vh, uint32_t &i) {
    const int h = t >= vh;
    i = (uint32_t)(t - h * vh);
    return p + (size_t)h * (24 / St<S>::W) * (size_t)padded_sites(vh);
}

template <typename S>
DEV void ld(const typename St<S>::vec *p, int t, int vh, double *o) {
    uint32_t i;
    const typename St<S>::vec *b = blk_base<S>(p, t, vh, i);
    typename St<S>::acc r[24];
    load_field<S, 24>(b, i, r);
#pragma unroll
    for (int k = 0; k < 24; ++k) o[k] = (double)r[k];
}
// The same load with a streaming hint: for the Krylov basis vectors, which a kernel reads once
// (so they do not push the vectors it writes and reads back out of L2).
template <typename S>
DEV void ld_basis(const typename St<S>::vec *p, int t, int vh, double *o) {
    uint32_t i;
    const typename St<S>::vec *b = blk_base<S>(p, t, vh, i);
    typename St<S>::acc r[24];
    load_planes_h<S, 24, true>(b, 24 / St<S>::W, 0, i, r);
#pragma unroll
    for (int k = 0; k < 24; ++k) o[k] = (double)r[k];
}
template <typename S>
DEV void st(typename St<S>::vec *p, int t, int vh, const double *o) {
    uint32_t i;
    typename St<S>::vec *b = blk_base<S>(p, t, vh, i);
    typename St<S>::acc r[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) r[k] = (typename St<S>::acc)o[k];
    store_field<S, 24>(b, i, r);
}

// Sum of v over the work-group (fixed tree: wave shuffles, then the waves in order).
template <int N>
DEV void group_sum(double v[N], double *lds /* [N][kRed / 64] */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < N; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) lds[k * (kRed / 64) + wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < kRed / 64; ++w) s += lds[k * (kRed / 64) + w];
            v[k] = s;
        }
    }
}

// A batch of nrhs independent systems: vector r of an argument v is v + r * vs (vs = the
// vector length in 16-byte units), basis vector j of system r is Q + (j * nrhs + r) * vs;
// system r's device scalars start r * sstride doubles after a scalar pointer.  Work-group b
// works on system b / nb; systems whose `active` flag is 0 are skipped entirely.
struct Bat {
    int n, vh, nb, nrhs, sstride;
    const int *active;
};

template <typename S>
DEV size_t vstride(const Bat &b) {
    return (size_t)(b.n / b.vh) * (24 / St<S>::W) * (size_t)padded_sites(b.vh);
}
DEV bool sys_of(const Bat &b, int &r, int &t) {
    r = blockIdx.x / b.nb;
    t = (blockIdx.x - r * b.nb) * kRed + threadIdx.x;
    return !b.active || b.active[r];
}

// partials[sys][blk] (complex) = sum over the group's sites of <a, b>
template <typename S>
__global__ __launch_bounds__(kRed) void k_dot(Bat B, const typename St<S>::vec *a, const typename St<S>::vec *b,
                                              double2 *partials) {
    __shared__ double lds[2 * kRed / 64];
    int r, t;
    if (!sys_of(B, r, t)) return;
    const size_t vs = vstride<S>(B);
    double v[2] = {0.0, 0.0};
    if (t < B.n) {
        double x[24], y[24];
        ld<S>(b + r * vs, t, B.vh, x);
        ld_basis<S>(a + r * vs, t, B.vh, y);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            v[0] = fma(y[2 * c], x[2 * c], v[0]);
            v[0] = fma(y[2 * c + 1], x[2 * c + 1], v[0]);
            v[1] = fma(y[2 * c], x[2 * c + 1], v[1]);
            v[1] = fma(-y[2 * c + 1], x[2 * c], v[1]);
        }
    }
    group_sum<2>(v, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = make_double2(v[0], v[1]);
}

// out_r = scale * sum_b partials[r][b] (b ascending), nc <= 2 doubles; one work-group per system
__global__ __launch_bounds__(kRed) void k_reduce(int nblk, int nc, const double *partials, double scale, double *out,
                                                 int sstride, const int *active) {
    __shared__ double lds[2 * kRed / 64];
    const int r = blockIdx.x;
    if (active && !active[r]) return;
    partials += (size_t)r * nblk * nc;
    double v[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < nblk; b += kRed)
        for (int c = 0; c < nc; ++c) v[c] += partials[(size_t)b * nc + c];
    group_sum<2>(v, lds);
    if (threadIdx.x == 0)
        for (int c = 0; c < nc; ++c) out[(size_t)r * sstride + c] = scale * v[c];
}

// ------------------------------------------------------------------ one GCR orthogonalisation step
// Two kernels per iteration, each finished by its last work-group per system, instead of a kernel and a
// reduction for each of the dots, the subtraction and the update, and one for the scalars; a third one corrects:
//   k_gcr_dots: <Q_j, q> (j < k), |q|^2 and <q, r> in one pass over Q, q and r; then beta_j = <Q_j, q> / |Q_j|^2,
//     gamma = |q|, and an estimate a of alpha: |q_perp|^2 = |q|^2 - sum_j |<Q_j, q>|^2 / |Q_j|^2 and <q_perp, r> = <q, r>
//     hold for orthogonal Q_j and r; a = 0 where less than a hundredth of |q|^2 is left by that;
//   k_gcr_step: Q_k = (q - sum_j beta_j Q_j) / gamma over q (k = 0: Q_0 = q, gamma = 1), r_new = r - a Q_k, and |Q_k|^2,
//     <Q_k, r>, |r_new|^2 of the vectors as stored; then alpha = <Q_k, r> / |Q_k|^2 is known;
//   k_gcr_correct: r_new -= (alpha - a) Q_k and |r_new|^2 anew, where |alpha - a|^2 |Q_k|^2 (what the estimate adds to the
//     least |r_new|^2) is above `slack` |r_new|^2, 1e-10 or what rounding the stored r adds; else alpha = a counts as
//     taken.  It follows every step of a batch, where it returns at once (3 to 5 us); a single solve leaves it out
//     until a step needs it (`defer`), which costs up to three iterations queued for nothing, once per solve.
// So the beta, the step and the solution's coefficients rest on sums over the stored vectors: the estimate
// cancels where q nearly lies in the span of the Q_j, and with alpha and gamma from it alone directions with
// |q_perp| / |q| below 1e-7 in FP64 (3e-5 in FP32) had to be left out, and solves that need one did not
// converge.  Here such a direction is taken with what is left of it, be it rounding (which leads out of a
// breakdown of GCR, where <r, A r> = 0).  Where nothing is left, Q_k = 0, the step is empty and the cycle ends.
// r_new goes to the next direction's slot (or over r): r is not stored a second time.  Passes over
// vectors per iteration: 2 k + 6 (5 for k = 0), against 2 k + 9; 2 k + 9 with a correction.
// Work-groups of k_gcr_dots and k_gcr_step take chunks of BS sites in turn, one site per thread; BS = 512, or 256
// where 512 would leave compute units without a work-group.  On the smallest lattices (kWideSites) a thread would
// still wait for one basis vector after the other (1.6 us each in FP64), so there (WIDE) a chunk is 64 sites and
// wavefront w of eight takes the basis vectors w, w + 8, ...: at 8^4 a kernel of an FP64 GCR(32) step falls from 34
// to 9 us on average; at 16^3 x 32 one right-hand side is slower that way (92 against 78 us per iteration).
// k_gcr_correct, which reads no basis vectors, takes one 16-byte vector per thread.  The partial sums and the
// finishing work-group's reads of them are agent-scope accesses (the XCDs' L2s are not coherent with each
// other), summed in a fixed order.
constexpr int kGcr = 512;
constexpr int kGcrBlocks = 512;  // work-groups per system at most: two per compute unit
constexpr int kGcrEnt = 2 * (64 + 2);
constexpr int kWideSites = 1 << 15;  // sites times systems

template <int CTRL, int ROWS>
DEV double dpp_part(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}
// sum over the wavefront in lane 63 (row shifts, then the rows in order)
DEV double wave_sum63(double v) {
    v += dpp_part<0x111, 0xf>(v);
    v += dpp_part<0x112, 0xf>(v);
    v += dpp_part<0x114, 0xf>(v);
    v += dpp_part<0x118, 0xf>(v);
    v += dpp_part<0x142, 0xa>(v);
    v += dpp_part<0x143, 0xc>(v);
    return v;
}

// A system's count of finished work-groups, zero between launches: a slot of its scalars.
DEV unsigned *gcr_count(double *scal) { return reinterpret_cast<unsigned *>(scal + S_COUNT); }

// Partial sums of a work-group, acc[wave][e] for e < ne, to part; true in every thread of the work-group that
// finishes last of the system's nblk, with tot[e] (in acc[0]) the sums over all of them.
template <int BS>
DEV bool gcr_finish(double (*acc)[kGcrEnt], int ne, int nblk, int sys, int blk, double *part, unsigned *ctr) {
    __shared__ bool last;
    constexpr int NW = BS / 64;
    const int tid = threadIdx.x;
    __syncthreads();
    part += (size_t)sys * nblk * ne;
    if (tid < ne) {
        double s = acc[0][tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += acc[w][tid];
        __hip_atomic_store(part + (size_t)blk * ne + tid, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial sums have arrived before the count goes up
    __syncthreads();
    if (tid == 0)
        last = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nblk - 1;
    __syncthreads();
    if (!last) return false;
    if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    double *flat = &acc[0][0];
    const int groups = BS / ne, g = tid / ne, e = tid - g * ne;
    double s = 0.0;
    if (g < groups) {
#pragma unroll 8
        for (int b = g; b < nblk; b += groups)
            s += __hip_atomic_load(part + (size_t)b * ne + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (g < groups) flat[g * ne + e] = s;
    __syncthreads();
    if (tid < ne) {
        for (int q = 1; q < groups; ++q) s += flat[q * ne + tid];
        flat[tid] = s;
    }
    __syncthreads();
    return true;
}

// The same for few sums that every thread holds a part of, v[e]: the totals are in v of thread 0 of the work-group
// that finishes last (which all of its threads are told).
template <int BS, int NE>
DEV bool gcr_finish_few(double (&v)[NE], int nblk, int sys, int blk, double *part, unsigned *ctr) {
    static_assert(kGcrBlocks <= 2 * BS, "two partial sums per thread at most");
    __shared__ double red[BS / 64][NE];
    __shared__ bool last;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    auto group = [&]() {  // v of thread 0 = sum over the work-group
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            v[e] = wave_sum63(v[e]);
            if (lane == 63) red[w][e] = v[e];
        }
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                v[e] = red[0][e];
#pragma unroll
                for (int u = 1; u < BS / 64; ++u) v[e] += red[u][e];
            }
        }
    };
    group();
    part += (size_t)sys * nblk * NE;
    if (tid == 0) {
#pragma unroll
        for (int e = 0; e < NE; ++e)
            __hip_atomic_store(part + (size_t)blk * NE + e, v[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial sums have arrived before the count goes up
        last = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nblk - 1;
    }
    __syncthreads();
    if (!last) return false;
    if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        v[e] = 0.0;
        for (int b = tid; b < nblk; b += BS)
            v[e] += __hip_atomic_load(part + (size_t)b * NE + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    group();
    return true;
}

// Back-substitution at the end of a cycle, one work-group per system: alpha_j = c_j gamma_j + sum_{k > j} c_k beta_kj,
// solved for c_{n-1} .. c_0 with one wavefront (lane j holds what is left of alpha_j), the beta in LDS.
// n = counts[sys], or n_all; c_j = 0 for n <= j < kmax.
__global__ __launch_bounds__(256) void k_gcr_backsub(const int *active, const int *counts, int n_all, int kmax,
                                                     int sstride, double *scal) {
    __shared__ double2 beta[kGcrMax * kGcrMax];
    const int sys = (int)blockIdx.x;
    if (active && !active[sys]) return;
    scal += (size_t)sys * sstride;
    const int n = counts ? counts[sys] : n_all;
    const double2 *bg = reinterpret_cast<const double2 *>(scal + S_BETA);
    for (int e = threadIdx.x; e < n * kGcrMax; e += 256) beta[e] = bg[e];  // entries j >= k are not used
    __syncthreads();
    const int lane = threadIdx.x;
    if (lane >= 64) return;
    double ar = 0.0, ai = 0.0, ig = 0.0;
    if (lane < n) {
        ar = scal[S_ALP + 2 * lane];
        ai = scal[S_ALP + 2 * lane + 1];
        ig = 1.0 / scal[S_GAM + lane];
    }
    for (int k = n - 1; k >= 0; --k) {
        const double cr = __shfl(ar * ig, k, 64), ci = __shfl(ai * ig, k, 64);
        if (lane < k) {
            const double2 b = beta[k * kGcrMax + lane];
            ar -= b.x * cr - b.y * ci;
            ai -= b.x * ci + b.y * cr;
        }
    }
    if (lane < kmax) {
        scal[S_C + 2 * lane] = lane < n ? ar * ig : 0.0;
        scal[S_C + 2 * lane + 1] = lane < n ? ai * ig : 0.0;
    }
}

template <typename S, bool WIDE, int BS>
__global__ __launch_bounds__(BS) void k_gcr_dots(Bat B, int nblk, const typename St<S>::vec *Q, int k,
                                                 const typename St<S>::vec *q, const typename St<S>::vec *rv, double *part,
                                                 double scale, double *scal) {
    __shared__ double acc[BS / 64][kGcrEnt];
    const int sys = (int)blockIdx.x / nblk, blk = (int)blockIdx.x - sys * nblk;
    if (B.active && !B.active[sys]) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, ne = 2 * k + 3;
    for (int e = lane; e < ne; e += 64) acc[w][e] = 0.0;
    const size_t vs = vstride<S>(B);
    q += sys * vs;
    rv += sys * vs;
    constexpr int CH = WIDE ? 64 : BS;
    const int nch = (B.n + CH - 1) / CH;
    for (int c = blk; c < nch; c += nblk) {
        const int t = c * CH + (WIDE ? lane : (int)threadIdx.x);
        const bool on = t < B.n;
        double a[24];
        if (on) ld<S>(q, t, B.vh, a);
        if (!WIDE || w == 0) {
            double v[3] = {0.0, 0.0, 0.0};
            if (on) {
                double b[24];
                ld<S>(rv, t, B.vh, b);
#pragma unroll
                for (int m = 0; m < 12; ++m) {
                    v[0] = fma(a[2 * m], a[2 * m], fma(a[2 * m + 1], a[2 * m + 1], v[0]));
                    v[1] = fma(a[2 * m], b[2 * m], fma(a[2 * m + 1], b[2 * m + 1], v[1]));
                    v[2] = fma(a[2 * m], b[2 * m + 1], fma(-a[2 * m + 1], b[2 * m], v[2]));
                }
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) v[m] = wave_sum63(v[m]);
            if (lane == 63) {
#pragma unroll
                for (int m = 0; m < 3; ++m) acc[w][2 * k + m] += v[m];
            }
        }
        for (int j = WIDE ? w : 0; j < k; j += WIDE ? (BS / 64) : 1) {
            double u[2] = {0.0, 0.0};
            if (on) {
                double b[24];
                ld_basis<S>(Q + ((size_t)j * B.nrhs + sys) * vs, t, B.vh, b);
#pragma unroll
                for (int m = 0; m < 12; ++m) {
                    u[0] = fma(b[2 * m], a[2 * m], fma(b[2 * m + 1], a[2 * m + 1], u[0]));
                    u[1] = fma(b[2 * m], a[2 * m + 1], fma(-b[2 * m + 1], a[2 * m], u[1]));
                }
            }
            u[0] = wave_sum63(u[0]);
            u[1] = wave_sum63(u[1]);
            if (lane == 63) {
                acc[w][2 * j] += u[0];
                acc[w][2 * j + 1] += u[1];
            }
        }
    }
    scal += (size_t)sys * B.sstride;
    if (!gcr_finish<BS>(acc, ne, nblk, sys, blk, part, gcr_count(scal))) return;
    if (w) return;
    // one wavefront: lane j forms beta_j
    const double *tot = acc[0];
    double sub = 0.0;
    if (lane < k) {
        const double n2 = scal[S_N2 + lane], inv = n2 > 0.0 ? 1.0 / n2 : 0.0;
        const double dr = scale * tot[2 * lane], di = scale * tot[2 * lane + 1];
        double *beta = scal + S_BETA + 2 * kGcrMax * k + 2 * lane;
        beta[0] = dr * inv;
        beta[1] = di * inv;
        sub = (dr * dr + di * di) * inv;
    }
    sub = wave_sum63(sub);
    if (lane == 63) {
        const double qq = scale * tot[2 * k], perp = qq - sub;
        const double g = k == 0 || qq == 0.0 ? 1.0 : sqrt(qq);  // NaN goes on into the step
        const double f = perp <= 0.01 * qq ? 0.0 : scale * g / perp;
        scal[S_SC] = 1.0 / g;
        scal[S_SC + 1] = f * tot[2 * k + 1];
        scal[S_SC + 2] = f * tot[2 * k + 2];
        scal[S_GAM + k] = g;
    }
}

// o rounded to the storage precision, stored, and returned as stored
template <typename S>
DEV void st_rounded(typename St<S>::vec *p, int t, int vh, double *o) {
    constexpr int W = St<S>::W;
    uint32_t i;
    typename St<S>::vec *q = site_ptr(blk_base<S>(p, t, vh, i), i, 24 / W);
#pragma unroll
    for (int m = 0; m < 24 / W; ++m) {
        typename St<S>::acc r[W];
#pragma unroll
        for (int e = 0; e < W; ++e) r[e] = (typename St<S>::acc)o[m * W + e];
        const typename St<S>::vec v = St<S>::pack(r);
        q[m * kSB] = v;
        St<S>::unpack(v, r);
#pragma unroll
        for (int e = 0; e < W; ++e) o[m * W + e] = (double)r[e];
    }
}

// Iteration control of a cycle (one system) after a step to the residual norm^2 rn2: ++ctl[1]; ctl[0] = 0 when the norm
// is at most target or not finite (then ctl[2] = 1), or when the step was empty.
DEV void gcr_control(int *ctl, double rn2, double target, bool empty) {
    ++ctl[1];
    if (!isfinite(rn2)) {
        ctl[2] = 1;
        ctl[0] = 0;
    } else if (sqrt(rn2) <= target || empty) {
        ctl[0] = 0;
    }
}

// WIDE: the wavefronts' parts of sum_j beta_j Q_j meet in LDS, and wavefront w then takes the storage planes
// w, w + 8 of the chunk's sites.
template <typename S, bool WIDE, int BS>
__global__ __launch_bounds__(BS) void k_gcr_step(Bat B, int nblk, const typename St<S>::vec *Q, int k,
                                                 typename St<S>::vec *q, const typename St<S>::vec *rv,
                                                 typename St<S>::vec *rnew, double *part, double scale, double slack,
                                                 double *scal, int *ctl, double target, int defer) {
    __shared__ double sub[WIDE ? (BS / 64) : 1][WIDE ? 24 : 1][64];
    const int sys = (int)blockIdx.x / nblk, blk = (int)blockIdx.x - sys * nblk;
    if (B.active && !B.active[sys]) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t vs = vstride<S>(B);
    q += sys * vs;
    rv += sys * vs;
    rnew += sys * vs;
    scal += (size_t)sys * B.sstride;
    const double2 *cf = reinterpret_cast<const double2 *>(scal + S_BETA + 2 * kGcrMax * k);
    const double ig = scal[S_SC], ar = scal[S_SC + 1], ai = scal[S_SC + 2];
    double v[4] = {0.0, 0.0, 0.0, 0.0};  // |Q_k|^2, <Q_k, r>, |r_new|^2
    auto dots = [&](double yr, double yi, double rr, double ri) {  // one complex component of Q_k and r
        v[0] = fma(yr, yr, fma(yi, yi, v[0]));
        v[1] = fma(yr, rr, fma(yi, ri, v[1]));
        v[2] = fma(yr, ri, fma(-yi, rr, v[2]));
    };
    constexpr int CH = WIDE ? 64 : BS;
    const int nch = (B.n + CH - 1) / CH;
    for (int c = blk; c < nch; c += nblk) {
        const int t = c * CH + (WIDE ? lane : (int)threadIdx.x);
        double a[24], b[24];
        auto take = [&](int j) {  // a -= beta_j Q_j
            const double2 cj = cf[j];
            ld_basis<S>(Q + ((size_t)j * B.nrhs + sys) * vs, t, B.vh, b);
#pragma unroll
            for (int m = 0; m < 12; ++m) {
                a[2 * m] -= cj.x * b[2 * m] - cj.y * b[2 * m + 1];
                a[2 * m + 1] -= cj.x * b[2 * m + 1] + cj.y * b[2 * m];
            }
        };
        if constexpr (!WIDE) {
            if (t >= B.n) continue;
            ld<S>(q, t, B.vh, a);
            if (k) {
                for (int j = 0; j < k; ++j) take(j);
#pragma unroll
                for (int m = 0; m < 24; ++m) a[m] *= ig;
                st_rounded<S>(q, t, B.vh, a);  // the stored (rounded) vector is what the recurrence uses
            }
            ld<S>(rv, t, B.vh, b);
#pragma unroll
            for (int m = 0; m < 12; ++m) {
                dots(a[2 * m], a[2 * m + 1], b[2 * m], b[2 * m + 1]);
                b[2 * m] -= ar * a[2 * m] - ai * a[2 * m + 1];
                b[2 * m + 1] -= ar * a[2 * m + 1] + ai * a[2 * m];
            }
            st_rounded<S>(rnew, t, B.vh, b);
#pragma unroll
            for (int m = 0; m < 24; ++m) v[3] = fma(b[m], b[m], v[3]);
        } else {
            constexpr int W = St<S>::W, NP = 24 / W;
            const int nw = min(k, (BS / 64));  // wavefronts with a basis vector
            if (w < nw) {
#pragma unroll
                for (int m = 0; m < 24; ++m) a[m] = 0.0;
                if (t < B.n)
                    for (int j = w; j < k; j += (BS / 64)) take(j);
#pragma unroll
                for (int m = 0; m < 24; ++m) sub[w][m][lane] = a[m];
            }
            __syncthreads();
            if (t < B.n) {
                uint32_t i;
                const size_t off = (size_t)(blk_base<S>(q, t, B.vh, i) - q);
                auto site = [&](auto *p) { return site_ptr(p + off, i, NP); };
                for (int pl = w; pl < NP; pl += (BS / 64)) {
                    typename St<S>::vec vq = site(q)[pl * kSB];
                    typename St<S>::acc f[W];
                    double y[W];
                    St<S>::unpack(vq, f);
                    if (k) {
#pragma unroll
                        for (int e = 0; e < W; ++e) {
                            double z = (double)f[e];
                            for (int u = 0; u < nw; ++u) z += sub[u][pl * W + e][lane];
                            f[e] = (typename St<S>::acc)(z * ig);
                        }
                        vq = St<S>::pack(f);
                        site(q)[pl * kSB] = vq;
                        St<S>::unpack(vq, f);  // the stored (rounded) vector is what the recurrence uses
                    }
#pragma unroll
                    for (int e = 0; e < W; ++e) y[e] = (double)f[e];
                    typename St<S>::vec vr = site(rv)[pl * kSB];
                    St<S>::unpack(vr, f);
#pragma unroll
                    for (int e = 0; e < W; e += 2) {
                        dots(y[e], y[e + 1], (double)f[e], (double)f[e + 1]);
                        const double re = (double)f[e] - (ar * y[e] - ai * y[e + 1]);
                        const double im = (double)f[e + 1] - (ar * y[e + 1] + ai * y[e]);
                        f[e] = (typename St<S>::acc)re;
                        f[e + 1] = (typename St<S>::acc)im;
                    }
                    vr = St<S>::pack(f);
                    site(rnew)[pl * kSB] = vr;
                    St<S>::unpack(vr, f);
#pragma unroll
                    for (int e = 0; e < W; ++e) v[3] = fma((double)f[e], (double)f[e], v[3]);
                }
            }
            __syncthreads();  // sub is read before the next chunk overwrites it
        }
    }
    if (!gcr_finish_few<BS>(v, nblk, sys, blk, part, gcr_count(scal))) return;
    if (threadIdx.x) return;
    const double n2 = scale * v[0], rn2 = scale * v[3];
    const bool empty = n2 == 0.0;
    const double f = empty ? 0.0 : scale / n2, er = empty ? 0.0 : ar, ei = empty ? 0.0 : ai;  // step taken, if not corrected
    const double dr = f * v[1] - er, di = f * v[2] - ei;
    const bool correct = (dr * dr + di * di) * n2 > slack * rn2;  // false for NaN
    scal[S_N2 + k] = n2;
    scal[S_ALP + 2 * k] = correct ? er + dr : er;
    scal[S_ALP + 2 * k + 1] = correct ? ei + di : ei;
    scal[S_SC + 3] = dr;
    scal[S_SC + 4] = di;
    scal[S_RED + 4] = rn2;
    scal[S_RED + 6] = empty ? 1.0 : 0.0;
    scal[S_RED + 7] = correct ? 1.0 : 0.0;
    if (ctl && !correct) {
        gcr_control(ctl, rn2, target, empty);
    } else if (ctl && defer) {  // the cycle waits for the correction
        ctl[3] = 1;
        ctl[0] = 0;
    }
}

// The vectors of a system are taken as they lie, 16 bytes a thread, kU loads of each in flight.
template <typename S>
__global__ __launch_bounds__(kGcr) void k_gcr_correct(Bat B, int nblk, const typename St<S>::vec *q,
                                                      typename St<S>::vec *rnew, double *part, double scale,
                                                      double *scal, int *ctl, double target) {
    using V = typename St<S>::vec;
    constexpr int W = St<S>::W, NP = 24 / W, kU = 4;
    const int sys = (int)blockIdx.x / nblk, blk = (int)blockIdx.x - sys * nblk;
    if (B.active && !B.active[sys]) return;
    scal += (size_t)sys * B.sstride;
    if (scal[S_RED + 7] == 0.0) return;
    const size_t vs = vstride<S>(B);
    q += sys * vs;
    rnew += sys * vs;
    const double dr = scal[S_SC + 3], di = scal[S_SC + 4];
    // (32 bits: a solve keeps more than nine vectors, so one has less than 2^31 of its 16-byte pieces)
    const uint32_t half = (uint32_t)NP * (uint32_t)padded_sites(B.vh), nv = (uint32_t)vs, step = (uint32_t)nblk * kGcr;
    double v[1] = {0.0};
    for (uint32_t e0 = (uint32_t)blk * kGcr + threadIdx.x; e0 < nv; e0 += kU * step) {
        V vq[kU], vr[kU];
        bool on[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t e = e0 + u * step, h = e >= half ? e - half : e;  // padding sites are left alone
            on[u] = e < nv && (h / (NP * kSB)) * kSB + (h & (kSB - 1)) < (uint32_t)B.vh;
            if (on[u]) {
                vq[u] = q[e];
                vr[u] = rnew[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (!on[u]) continue;
            typename St<S>::acc y[W], f[W];
            St<S>::unpack(vq[u], y);
            St<S>::unpack(vr[u], f);
#pragma unroll
            for (int c = 0; c < W; c += 2) {
                const double yr = (double)y[c], yi = (double)y[c + 1];
                const double re = (double)f[c] - (dr * yr - di * yi), im = (double)f[c + 1] - (dr * yi + di * yr);
                f[c] = (typename St<S>::acc)re;
                f[c + 1] = (typename St<S>::acc)im;
            }
            const V o = St<S>::pack(f);
            rnew[e0 + u * step] = o;
            St<S>::unpack(o, f);
#pragma unroll
            for (int c = 0; c < W; ++c) v[0] = fma((double)f[c], (double)f[c], v[0]);
        }
    }
    if (!gcr_finish_few<kGcr>(v, nblk, sys, blk, part, gcr_count(scal))) return;
    if (threadIdx.x) return;
    const double rn2 = scale * v[0];
    scal[S_RED + 4] = rn2;
    if (ctl) {
        ctl[3] = 0;
        ctl[0] = 1;
        gcr_control(ctl, rn2, target, false);
    }
}

// x += xscale_r sum_j coef_j P_j (x and P may have different precisions)
template <typename SX, typename SP>
__global__ __launch_bounds__(kRed) void k_axpy_multi(Bat B, typename St<SX>::vec *x, const typename St<SP>::vec *P,
                                                     int k, const double *coef, double xscale,
                                                     const double *xscales, const int *kcount) {
    int r, t;
    if (!sys_of(B, r, t) || t >= B.n) return;
    x += r * vstride<SX>(B);
    const size_t vp = vstride<SP>(B);
    const double2 *cf = reinterpret_cast<const double2 *>(coef + (size_t)r * B.sstride);
    const double xs = xscales ? xscales[(size_t)r * B.sstride] : xscale;
    // a system's own count of basis vectors: those past it were not written in this cycle
    const int kr = kcount ? min(k, kcount[r]) : k;
    double a[24], b[24];
    ld<SX>(x, t, B.vh, a);
    for (int j = 0; j < kr; ++j) {
        const double2 cj = cf[j];
        ld_basis<SP>(P + ((size_t)j * B.nrhs + r) * vp, t, B.vh, b);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            a[2 * c] += xs * (cj.x * b[2 * c] - cj.y * b[2 * c + 1]);
            a[2 * c + 1] += xs * (cj.x * b[2 * c + 1] + cj.y * b[2 * c]);
        }
    }
    st<SX>(x, t, B.vh, a);
}

// out = alpha_r a + beta b (converted to the output precision); optional copy2 = out; partial |out|^2
// and a non-finite flag.  alpha_r = alphas[r * sstride] when alphas is given.
template <typename SO, typename SA, typename SB>
__global__ __launch_bounds__(kRed) void k_lincomb(Bat B, typename St<SO>::vec *out, typename St<SO>::vec *copy2,
                                                  double alpha, const double *alphas, const typename St<SA>::vec *a,
                                                  double beta, const typename St<SB>::vec *b, double *partials) {
    __shared__ double lds[2 * kRed / 64];
    int r, t;
    if (!sys_of(B, r, t)) return;
    out += r * vstride<SO>(B);
    if (copy2) copy2 += r * vstride<SO>(B);
    a += r * vstride<SA>(B);
    if (b) b += r * vstride<SB>(B);
    const double al = alphas ? alphas[(size_t)r * B.sstride] : alpha;
    double v[2] = {0.0, 0.0};
    if (t < B.n) {
        double x[24], y[24];
        ld<SA>(a, t, B.vh, x);
        if (b) {
            ld<SB>(b, t, B.vh, y);
#pragma unroll
            for (int c = 0; c < 24; ++c) x[c] = al * x[c] + beta * y[c];
        } else {
#pragma unroll
            for (int c = 0; c < 24; ++c) x[c] = al * x[c];
        }
        st<SO>(out, t, B.vh, x);
        if (copy2) st<SO>(copy2, t, B.vh, x);
        bool fin = true;
#pragma unroll
        for (int c = 0; c < 24; ++c) {
            v[0] += x[c] * x[c];
            fin = fin && isfinite(x[c]);
        }
        v[1] = fin ? 0.0 : 1.0;
    }
    if (partials) {
        group_sum<2>(v, lds);
        if (threadIdx.x == 0) {
            partials[(size_t)blockIdx.x * 2] = v[0];
            partials[(size_t)blockIdx.x * 2 + 1] = v[1];
        }
    }
}

// CG-style update for CGLS: x += alpha p; s -= alpha w (alpha = num / den from device scalars)
template <typename S>
__global__ __launch_bounds__(kRed) void k_cgls_xs(int n, int vh, const double *rho, const double *wn,
                                                  typename St<S>::vec *x, const typename St<S>::vec *p,
                                                  typename St<S>::vec *s, const typename St<S>::vec *w,
                                                  double *partials) {
    __shared__ double lds[kRed / 64];
    const int t = blockIdx.x * kRed + threadIdx.x;
    double v[1] = {0.0};
    if (t < n) {
        const double alpha = rho[0] / wn[0];
        double a[24], b[24];
        ld<S>(x, t, vh, a);
        ld<S>(p, t, vh, b);
#pragma unroll
        for (int c = 0; c < 24; ++c) a[c] += alpha * b[c];
        st<S>(x, t, vh, a);
        ld<S>(s, t, vh, a);
        ld<S>(w, t, vh, b);
#pragma unroll
        for (int c = 0; c < 24; ++c) {
            a[c] -= alpha * b[c];
            v[0] += a[c] * a[c];
        }
        st<S>(s, t, vh, a);
    }
    group_sum<1>(v, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

// p = r + (rho_new / rho_old) p
template <typename S>
__global__ __launch_bounds__(kRed) void k_cgls_p(int n, int vh, const double *rho_new, const double *rho_old,
                                                 typename St<S>::vec *p, const typename St<S>::vec *r) {
    const int t = blockIdx.x * kRed + threadIdx.x;
    if (t >= n) return;
    const double beta = rho_new[0] / rho_old[0];
    double a[24], b[24];
    ld<S>(p, t, vh, a);
    ld<S>(r, t, vh, b);
#pragma unroll
    for (int c = 0; c < 24; ++c) a[c] = b[c] + beta * a[c];
    st<S>(p, t, vh, a);
}

__global__ void k_set(double *p, double v) {
    if (threadIdx.x == 0 && blockIdx.x == 0) p[0] = v;
}
__global__ void k_copy_scalar(const double *src, double *dst) {
    if (threadIdx.x == 0 && blockIdx.x == 0) dst[0] = src[0];
}

}  // namespace

// ------------------------------------------------------------------ host wrappers
int blas_grid(int64_t nsites) { return (int)((nsites + kRed - 1) / kRed); }

#define DISPATCH_PREC(pr, FN)                                                              \
    switch (pr) {                                                                          \
        case DIRAC_F64: FN(double); break;                                                 \
        case DIRAC_F32: FN(float); break;                                                  \
        case DIRAC_F16: FN(__half); break;                                                 \
        case DIRAC_BF16: FN(__hip_bfloat16); break;                                        \
        default: throw Error(DIRAC_EINVAL, "unknown precision");                           \
    }

void Blas::reserve(int64_t nsites_max, int nrhs) {
    nrhs = std::max(nrhs, 1);
    // the partial sums of the reductions by k_reduce, or of the GCR kernels
    part.alloc((size_t)nrhs * std::max<size_t>(2 * (size_t)blas_grid(nsites_max), kGcrBlocks * kGcrEnt) * sizeof(double));
    const size_t n = (size_t)nrhs * kSysScal;
    if (scal.bytes < n * sizeof(double)) {
        scal.alloc(n * sizeof(double));
        // zeros (S_COUNT) that have arrived when this returns: solves run on streams that do not wait for the null
        // stream, as a hipMemset would need
        const std::vector<double> zero(n, 0.0);
        HIP_CHECK(hipMemcpy(scal.p, zero.data(), n * sizeof(double), hipMemcpyHostToDevice));
    }
}

namespace {
Bat make_bat(const dirac_ctx *c, int nh, const BatchSpec &bs) {
    Bat b;
    b.vh = (int)c->vh;
    b.n = nh * b.vh;
    b.nb = blas_grid(b.n);
    b.nrhs = bs.nrhs;
    b.sstride = bs.sstride;
    b.active = bs.active;
    return b;
}
}  // namespace

void Blas::dot(dirac_prec pr, int nh, const void *x, const void *y, double *out_dev, double scale, hipStream_t s,
               const BatchSpec &bs) {
    const Bat b = make_bat(c, nh, bs);
#define FN(S)                                                                                                     \
    k_dot<S><<<b.nb * b.nrhs, kRed, 0, s>>>(b, (const typename St<S>::vec *)x, (const typename St<S>::vec *)y,     \
                                            (double2 *)part.p);
    DISPATCH_PREC(pr, FN)
#undef FN
    k_reduce<<<b.nrhs, kRed, 0, s>>>(b.nb, 2, (const double *)part.p, scale, out_dev, b.sstride, b.active);
    HIP_CHECK(hipGetLastError());
}

namespace {
// |r|^2 gains about u^2 / 4 |r|^2 when r is rounded to the storage (relative steps of at most u, uniform): 4e-6 in BF16
double gcr_slack(dirac_prec pr) {
    const double u = pr == DIRAC_F16 ? 0x1p-11 : pr == DIRAC_BF16 ? 0x1p-8 : 0.0;
    return std::max(1e-10, 0.25 * u * u);
}
bool gcr_wide(const Bat &b) { return (int64_t)b.n * b.nrhs <= kWideSites; }
int gcr_block_size(const Bat &b) { return gcr_wide(b) || (int64_t)b.n * b.nrhs >= 256 * kGcr ? kGcr : kGcr / 2; }
int gcr_blocks(const Bat &b) {
    const int ch = gcr_wide(b) ? 64 : gcr_block_size(b);
    return std::min((b.n + ch - 1) / ch, kGcrBlocks);
}
}  // namespace

void Blas::gcr_dots(dirac_prec pr, int nh, const void *Q, int k, const void *q, const void *r, double scale,
                    hipStream_t s, const BatchSpec &bs) {
    const Bat b = make_bat(c, nh, bs);
    const int nblk = gcr_blocks(b);
#define FNW(S, WIDE, BS)                                                                                                \
    k_gcr_dots<S, WIDE, BS><<<nblk * b.nrhs, BS, 0, s>>>(b, nblk, (const typename St<S>::vec *)Q, k,                   \
                                                         (const typename St<S>::vec *)q,                               \
                                                         (const typename St<S>::vec *)r, (double *)part.p, scale, (double *)scal.p);
#define FN(S) if (gcr_wide(b)) { FNW(S, true, kGcr) } else if (gcr_block_size(b) == kGcr) { FNW(S, false, kGcr) } else { FNW(S, false, kGcr / 2) }
    DISPATCH_PREC(pr, FN)
#undef FN
#undef FNW
    HIP_CHECK(hipGetLastError());
}

void Blas::gcr_backsub(const int *counts, int n, int kmax, hipStream_t s, const BatchSpec &bs) {
    k_gcr_backsub<<<bs.nrhs, 256, 0, s>>>(bs.active, counts, n, kmax, bs.sstride, (double *)scal.p);
    HIP_CHECK(hipGetLastError());
}

void Blas::gcr_step(dirac_prec pr, int nh, const void *Q, int k, void *q, const void *r, void *rnew, double scale,
                    hipStream_t s, const BatchSpec &bs, int *ctl, double target, bool defer) {
    const Bat b = make_bat(c, nh, bs);
    const int nblk = gcr_blocks(b);
#define FNW(S, WIDE, BS)                                                                                              \
    k_gcr_step<S, WIDE, BS><<<nblk * b.nrhs, BS, 0, s>>>(b, nblk, (const typename St<S>::vec *)Q, k,                 \
                                                         (typename St<S>::vec *)q, (const typename St<S>::vec *)r,   \
                                                         (typename St<S>::vec *)rnew, (double *)part.p, scale,       \
                                                         gcr_slack(pr), (double *)scal.p, ctl, target, defer ? 1 : 0);
#define FN(S) if (gcr_wide(b)) { FNW(S, true, kGcr) } else if (gcr_block_size(b) == kGcr) { FNW(S, false, kGcr) } else { FNW(S, false, kGcr / 2) }
    DISPATCH_PREC(pr, FN)
#undef FN
#undef FNW
    HIP_CHECK(hipGetLastError());
    if (!defer) gcr_correct(pr, nh, q, rnew, scale, s, bs, ctl, target);
}

void Blas::gcr_correct(dirac_prec pr, int nh, const void *q, void *rnew, double scale, hipStream_t s,
                       const BatchSpec &bs, int *ctl, double target) {
    const Bat b = make_bat(c, nh, bs);
    const int64_t nv = (int64_t)(b.n / b.vh) * (24 * real_size(pr) / 16) * padded_sites(b.vh);  // 16-byte vectors
    // rarely with work: about one work-group per compute unit over all systems, so that the others' kernels do not
    // hold it up for long (3,072 of them took 90 us to return among the lattices of a batch)
    const int nr = (int)std::min<int64_t>((nv + kGcr - 1) / kGcr, std::max(kGcrBlocks / 2 / b.nrhs, 16));
#define FN(S)                                                                                                         \
    k_gcr_correct<S><<<nr * b.nrhs, kGcr, 0, s>>>(b, nr, (const typename St<S>::vec *)q, (typename St<S>::vec *)rnew, \
                                                  (double *)part.p, scale, (double *)scal.p, ctl, target);
    DISPATCH_PREC(pr, FN)
#undef FN
    HIP_CHECK(hipGetLastError());
}

void Blas::axpy_multi(dirac_prec px, dirac_prec pp, int nh, void *x, const void *P, int k, const double *coef_dev,
                      double xscale, hipStream_t s, const BatchSpec &bs, const double *xscales, const int *kcount) {
    const Bat b = make_bat(c, nh, bs);
#define FN2(SX, SP)                                                                                              \
    k_axpy_multi<SX, SP><<<b.nb * b.nrhs, kRed, 0, s>>>(b, (typename St<SX>::vec *)x,                             \
                                                        (const typename St<SP>::vec *)P, k, coef_dev, xscale,     \
                                                        xscales, kcount);
#define FN(SP)                                                                                     \
    if (px == DIRAC_F64) { FN2(double, SP) } else if (px == DIRAC_F32) { FN2(float, SP) }          \
    else if (px == DIRAC_F16) { FN2(__half, SP) } else { FN2(__hip_bfloat16, SP) }
    DISPATCH_PREC(pp, FN)
#undef FN
#undef FN2
    HIP_CHECK(hipGetLastError());
}

// out = alpha a + beta b (b may be NULL), copy2 = out if given; writes scale |out|^2 and a
// non-finite flag into out_dev[0..1] when out_dev is given.
void Blas::lincomb(dirac_prec po, dirac_prec pa, dirac_prec pb, int nh, void *out, void *copy2, double alpha,
                   const void *a, double beta, const void *b, double *out_dev, double scale, hipStream_t s,
                   const BatchSpec &bs, const double *alphas) {
    const Bat bt = make_bat(c, nh, bs);
    double *pp = out_dev ? (double *)part.p : nullptr;
#define FN3(SO, SA, SB)                                                                                           \
    k_lincomb<SO, SA, SB><<<bt.nb * bt.nrhs, kRed, 0, s>>>(bt, (typename St<SO>::vec *)out,                       \
                                                           (typename St<SO>::vec *)copy2, alpha, alphas,          \
                                                           (const typename St<SA>::vec *)a, beta,                 \
                                                           (const typename St<SB>::vec *)b, pp);
    if (po == pa && pa == pb) {
#define FN(S) FN3(S, S, S)
        DISPATCH_PREC(po, FN)
#undef FN
    } else if (pa == DIRAC_F64 && pb == DIRAC_F64) {
#define FN(S) FN3(S, double, double)
        DISPATCH_PREC(po, FN)
#undef FN
    } else if (po == DIRAC_F64 && pb == DIRAC_F64) {
#define FN(S) FN3(double, S, double)
        DISPATCH_PREC(pa, FN)
#undef FN
    } else {
        throw Error(DIRAC_EUNSUPPORTED, "lincomb precision combination");
    }
#undef FN3
    if (out_dev)
        k_reduce<<<bt.nrhs, kRed, 0, s>>>(bt.nb, 2, (const double *)part.p, scale, out_dev, bt.sstride, bt.active);
    HIP_CHECK(hipGetLastError());
}

void Blas::cgls_xs(int nh, const double *rho, const double *wn, void *x, const void *p, void *sv, const void *w,
                   double *out_dev, hipStream_t s) {
    const int vh = (int)c->vh, n = nh * vh, nb = blas_grid(n);
    k_cgls_xs<double><<<nb, kRed, 0, s>>>(n, vh, rho, wn, (double2 *)x, (const double2 *)p, (double2 *)sv,
                                          (const double2 *)w, (double *)part.p);
    k_reduce<<<1, kRed, 0, s>>>(nb, 1, (const double *)part.p, 1.0, out_dev, 0, nullptr);
    HIP_CHECK(hipGetLastError());
}

void Blas::cgls_p(int nh, const double *rho_new, const double *rho_old, void *p, const void *r, hipStream_t s) {
    const int vh = (int)c->vh, n = nh * vh, nb = blas_grid(n);
    k_cgls_p<double><<<nb, kRed, 0, s>>>(n, vh, rho_new, rho_old, (double2 *)p, (const double2 *)r);
    HIP_CHECK(hipGetLastError());
}

void Blas::set(double *p, double v, hipStream_t s) {
    k_set<<<1, 1, 0, s>>>(p, v);
    HIP_CHECK(hipGetLastError());
}
void Blas::copy_scalar(const double *src, double *dst, hipStream_t s) {
    k_copy_scalar<<<1, 1, 0, s>>>(src, dst);
    HIP_CHECK(hipGetLastError());
}

}  // namespace dl
