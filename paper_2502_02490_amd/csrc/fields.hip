// Field import and export: the user layouts of the boundary (LEX and EO site order,
// array-of-structs, paper Sec. 4.1) to and from the library's per-parity plane
// layout, link compression, and lower-precision copies of the operator fields.
#include <cstring>

#include "dirac_ops.h"
#include "internal.h"

namespace dl {
namespace {

// ------------------------------------------------------------------ links
// The LEX gauge field [V][4][9] as planes, per parity and direction [block][9][64 sites] of complex
// numbers, from which the clover field and the compressed links are built with coalesced reads.
// 128 consecutive LEX sites are the 64 even and 64 odd sites of one site block: they are read as they
// lie (72 KB, in four pieces of one direction each) and go through LDS; the angles follow in planes of
// reals.  Bandwidth-bound: 1216 B per site; 0.22 ms at 24^3 x 48 (3.7 TB/s).
__global__ __launch_bounds__(kBlock) void k_link_planes(Geom g, const double2 *__restrict__ U,
                                                        const double *__restrict__ theta,
                                                        double2 *__restrict__ planes, double *__restrict__ tp) {
    __shared__ double2 t[2 * kSB * 9];
    const int i0 = (int)blockIdx.x * kSB;
    const int ns = 2 * min(kSB, g.vh - i0);  // sites of this block
    const int lane = threadIdx.x & (kSB - 1), w = threadIdx.x >> 6;
    // LDS site of (parity, lane): sites 2 i and 2 i + 1, the one of that parity
    int x[4];
    site_coords(g, min(i0 + lane, g.vh - 1), 0, x);
    const int odd = x[3] & 1;
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
        for (int k = threadIdx.x; k < ns * 9; k += kBlock) t[k] = ld_stream(U + ((size_t)(2 * i0 + k / 9) * 4 + mu) * 9 + k % 9);
        __syncthreads();
        if (2 * lane < ns) {
            for (int k = w; k < 18; k += kBlock / kSB) {
                const int p = k / 9, e = k % 9;
                double2 *dst = site_ptr(planes + (size_t)(4 * p + mu) * 9 * g.vhp, (uint32_t)(i0 + lane), 9);
                dst[e * kSB] = t[(2 * lane + (odd ^ p)) * 9 + e];
            }
        }
        __syncthreads();
    }
    if (!theta || 2 * lane >= ns) return;
    for (int k = w; k < 8; k += kBlock / kSB)
        tp[(size_t)k * g.vhp + i0 + lane] = theta[((size_t)2 * i0 + 2 * lane + (odd ^ (k >> 2))) * 4 + (k & 3)];
}

// For site x of parity p (half index i) and direction mu:
//   dir 2 mu     : U_mu(x),        omega = qhat theta_mu(x) + phi_mu [x_mu = L_mu - 1]
//   dir 2 mu + 1 : U_mu(x - mu),   omega of that link (its x_mu is L_mu - 1 when x_mu = 0)
// Rows 0 and 1 of U are stored; row 2 is rebuilt as conj(row0 x row1) where used.
__global__ __launch_bounds__(kBlock) void k_import_links(Geom g, int p, const double2 *__restrict__ U,
                                                          const double *__restrict__ theta, int qhat,
                                                          double4 phase, double2 *__restrict__ planes,
                                                          double *__restrict__ omega,
                                                          unsigned long long *__restrict__ maxdev) {
    int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.vh) return;
    int x[4];
    site_coords(g, i, p, x);
    const double ph[4] = {phase.x, phase.y, phase.z, phase.w};
    const size_t vhp = (size_t)g.vhp;
    double dev = 0.0;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
#pragma unroll
        for (int back = 0; back < 2; ++back) {
            int y[4] = {x[0], x[1], x[2], x[3]};
            if (back) {
                const bool cross = y[mu] == 0;
                y[mu] = wrap_dn(y[mu], g.L[mu]);
                y[1] = cstar_x1(g, mu, cross, y[1]);  // C*: the link behind x may sit in the mirror copy
            }
            const int n = 4 * (p ^ back) + mu, j = half_index(g, y);
            const double2 *u = site_ptr(U + (size_t)n * 9 * vhp, (uint32_t)j, 9);
            const int dir = 2 * mu + back;
            double2 *dst = site_ptr(planes + (size_t)dir * 6 * vhp, (uint32_t)i, 6);
#pragma unroll
            for (int k = 0; k < 6; ++k) dst[k * kSB] = u[k * kSB];
            double w = (theta ? qhat * theta[n * vhp + j] : 0.0) + (y[mu] == g.L[mu] - 1 ? ph[mu] : 0.0);
            omega[(size_t)dir * vhp + i] = w;
            if (!back) {
                // deviation from SU(3): max |U U^dag - 1| and |det U - 1|; the row-2 rebuild needs det U = 1
                cx<double> m[9];
#pragma unroll
                for (int k = 0; k < 9; ++k) m[k] = mk(u[k * kSB].x, u[k * kSB].y);
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        cx<double> s = mk(0.0, 0.0);
#pragma unroll
                        for (int k = 0; k < 3; ++k) s = s + m[3 * a + k] * conj(m[3 * b + k]);
                        if (a == b) s.r -= 1.0;
                        dev = fmax(dev, fabs(s.r) + fabs(s.i));
                    }
                cx<double> det = m[0] * (m[4] * m[8] - m[5] * m[7]) - m[1] * (m[3] * m[8] - m[5] * m[6]) +
                                 m[2] * (m[3] * m[7] - m[4] * m[6]);
                dev = fmax(dev, fabs(det.r - 1.0) + fabs(det.i));
            }
        }
    }
    if (!(dev <= 1e300)) dev = 1e300;  // NaN input
    atomicMax(maxdev, (unsigned long long)__double_as_longlong(dev));
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_convert_links(int vh, int vhp, const double2 *__restrict__ src,
                                                           const double *__restrict__ om_src,
                                                           typename Lk<S>::vec *__restrict__ dst,
                                                           typename Lk<S>::om *__restrict__ om_dst) {
    int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= vh) return;
    constexpr int W = Lk<S>::W;
    const size_t n = (size_t)vhp;
    for (int dir = 0; dir < 8; ++dir) {
        double r[12];
        const double2 *s0 = site_ptr(src + (size_t)dir * 6 * n, (uint32_t)i, 6);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            double2 v = s0[k * kSB];
            r[2 * k] = v.x;
            r[2 * k + 1] = v.y;
        }
        typename Lk<S>::vec *d0 = site_ptr(dst + (size_t)dir * (12 / W) * n, (uint32_t)i, 12 / W);
#pragma unroll
        for (int k = 0; k < 12 / W; ++k) d0[k * kSB] = Lk<S>::pack(r + k * W);
        if constexpr (Lk<S>::phase_pair) {
            double si, co;
            sc(om_src[(size_t)dir * n + i], si, co);  // FP64, then rounded once to the 16-bit format
            om_dst[(size_t)dir * n + i] = Lk<S>::pack_phase((float)co, (float)si);
        } else {
            om_dst[(size_t)dir * n + i] = (typename Lk<S>::om)om_src[(size_t)dir * n + i];
        }
    }
}

// ------------------------------------------------------------------ clover (72 reals per site)
template <typename S>
__global__ __launch_bounds__(kBlock) void k_convert_clover(int vh, const double2 *__restrict__ src,
                                                            typename St<S>::vec *__restrict__ dst) {
    int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= vh) return;
    double r[72];
    load_field<double, 72>(src, i, r);
    typename St<S>::acc a[72];
#pragma unroll
    for (int k = 0; k < 72; ++k) a[k] = (typename St<S>::acc)r[k];
    store_field<S, 72>(dst, i, a);
}

// user index of the site (p, i): LEX -> Lambda, EO -> xhat, OPENQXD -> eq. (ipt) with the cache
// block (relative to the first site of the parity for half vectors)
DEV int64_t user_site(const Geom &g, int p, int i, int lay, int half) {
    if (lay == DIRAC_LAYOUT_LEX || lay == DIRAC_LAYOUT_OPENQXD) {
        int x[4];
        site_coords(g, i, p, x);
        if (lay == DIRAC_LAYOUT_LEX) return lex_index(g, x);
        const int64_t k = ipt_index(g, x);
        return half ? k - (int64_t)p * g.vh : k;
    }
    return half ? (int64_t)i : (int64_t)i + (int64_t)p * g.vh;
}

// Site fields of NR reals between the caller's order (NR consecutive reals per site) and the planes.  A work-group
// takes one 64-site block, both parities one after the other (in LEX order their sites alternate, so the
// cache lines of one are still in L2 for the other): the caller's side is accessed with consecutive lanes on
// consecutive reals of a site, the planes 1 KB at a time, and the block goes through LDS in between (an odd
// row length in reals: no bank conflicts either way).  Bandwidth-bound; one thread per site on both sides
// left the caller's side with 192 or 576 bytes between lanes.  On the way in a thread issues six or nine loads
// before it waits for the first (one at a time was slower than one thread per site for clover fields and for
// FP32 vectors in EO order).  One thread per site -> now: a LEX vector of 40 x 18 x 22 x 26 in FP64 in 33 -> 26 us, out
// 42 -> 25 us; an FP32 vector of 64 x 32^3 in EO order in 78 -> 70 us; a LEX clover field of 24^3 x 48 in 167 -> 145 us,
// out 219 -> 168 us (764 MB: the rate of a copy).
template <typename U, typename S, int NR>
__global__ __launch_bounds__(kBlock) void k_site_in(Geom g, int p0, int np, int lay, int half, const U *__restrict__ user,
                                                     typename St<S>::vec *__restrict__ dst0,
                                                     typename St<S>::vec *__restrict__ dst1) {
    using T = typename St<S>::acc;
    constexpr int W = St<S>::W, NP = NR / W;
    constexpr int IT = NR * kSB / kBlock, NB = IT % 9 == 0 ? 9 : 6;  // reals per thread, loaded NB at a time
    static_assert(NR * kSB % kBlock == 0 && IT % NB == 0, "whole batches of loads");
    __shared__ T t[kSB * (NR + 1)];
    __shared__ int64_t us[kSB];
    const int i0 = (int)blockIdx.x * kSB, ns = min(kSB, g.vh - i0), lane = threadIdx.x & (kSB - 1);
    for (int p = p0; p < p0 + np; ++p) {
        if (threadIdx.x < ns) us[threadIdx.x] = user_site(g, p, i0 + (int)threadIdx.x, lay, half) * NR;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < IT; b += NB) {
            U v[NB];
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                const int k = threadIdx.x + (b + e) * kBlock;
                if (k < ns * NR) v[e] = user[us[k / NR] + k % NR];
            }
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                const int k = threadIdx.x + (b + e) * kBlock;
                if (k < ns * NR) t[k + k / NR] = (T)v[e];
            }
        }
        __syncthreads();
        if (lane < ns) {
            typename St<S>::vec *q = site_ptr(p == p0 ? dst0 : dst1, (uint32_t)(i0 + lane), NP);
            for (int m = threadIdx.x >> 6; m < NP; m += kBlock / kSB) q[m * kSB] = St<S>::pack(t + lane * (NR + 1) + m * W);
        }
    }
}

template <typename U, typename S, int NR>
__global__ __launch_bounds__(kBlock) void k_site_out(Geom g, int p0, int np, int lay, int half,
                                                      const typename St<S>::vec *__restrict__ src0,
                                                      const typename St<S>::vec *__restrict__ src1, U *__restrict__ user) {
    using T = typename St<S>::acc;
    constexpr int W = St<S>::W, NP = NR / W;
    __shared__ T t[kSB * (NR + 1)];
    __shared__ int64_t us[kSB];
    const int i0 = (int)blockIdx.x * kSB, ns = min(kSB, g.vh - i0), lane = threadIdx.x & (kSB - 1);
    for (int p = p0; p < p0 + np; ++p) {
        const typename St<S>::vec *src = p == p0 ? src0 : src1;  // NULL: zeros
        if (threadIdx.x < ns) us[threadIdx.x] = user_site(g, p, i0 + (int)threadIdx.x, lay, half) * NR;
        if (lane < ns && src) {
            const typename St<S>::vec *q = site_ptr(src, (uint32_t)(i0 + lane), NP);
            for (int m = threadIdx.x >> 6; m < NP; m += kBlock / kSB)
                St<S>::unpack(q[m * kSB], t + lane * (NR + 1) + m * W);
        }
        __syncthreads();
        for (int k = threadIdx.x; k < ns * NR; k += kBlock) user[us[k / NR] + k % NR] = src ? (U)t[k + k / NR] : U(0);
        __syncthreads();
    }
}

template <typename S>
void convert_fields(dirac_ctx *c, dirac_prec pr, hipStream_t s) {
    PrecFields &lo = c->f[pr];
    PrecFields &hi = c->f[DIRAC_F64];
    const int vh = (int)c->vh;
    const size_t vhp = (size_t)c->g.vhp;
    if (!lo.links_ready) {
        for (int p = 0; p < 2; ++p) {
            lo.links[p].alloc_field((size_t)8 * 12 * sizeof(typename Lk<S>::vec) / Lk<S>::W * vhp);
            lo.omega[p].alloc_field((size_t)8 * sizeof(typename Lk<S>::om) * vhp);
            k_convert_links<S><<<grid_for(vh), kBlock, 0, s>>>(
                vh, (int)vhp, (const double2 *)hi.links[p].p, (const double *)hi.omega[p].p,
                (typename Lk<S>::vec *)lo.links[p].p, (typename Lk<S>::om *)lo.omega[p].p);
        }
        HIP_CHECK(hipGetLastError());
        lo.links_ready = true;
    }
    if (!lo.clover_ready) {
        for (int p = 0; p < 2; ++p) {
            lo.clov[p].alloc_field((size_t)72 * sizeof(S) * vhp);
            k_convert_clover<S><<<grid_for(vh), kBlock, 0, s>>>(vh, (const double2 *)hi.clov[p].p,
                                                                  (typename St<S>::vec *)lo.clov[p].p);
        }
        HIP_CHECK(hipGetLastError());
        lo.clover_ready = true;
    }
    for (int p = 0; p < 2; ++p) {
        if (hi.inv_ready[p] && !lo.inv_ready[p]) {
            lo.clinv[p].alloc_field((size_t)72 * sizeof(S) * vhp);
            k_convert_clover<S><<<grid_for(vh), kBlock, 0, s>>>(vh, (const double2 *)hi.clinv[p].p,
                                                                  (typename St<S>::vec *)lo.clinv[p].p);
            HIP_CHECK(hipGetLastError());
            lo.inv_ready[p] = true;
        }
    }
}

template <typename U, typename S>
void spinor_io(dirac_ctx *c, void *native, const void *user, bool in, int sites, dirac_layout lay, hipStream_t s) {
    using V = typename St<S>::vec;
    const size_t pv = (size_t)(24 / St<S>::W) * c->g.vhp;  // vectors of a parity
    const int nb = c->g.vhp / kSB, p0 = sites == 2, np = sites == 0 ? 2 : 1, half = sites != 0;
    if (in)
        k_site_in<U, S, 24><<<nb, kBlock, 0, s>>>(c->g, p0, np, lay, half, (const U *)user, (V *)native, (V *)native + pv);
    else
        k_site_out<U, S, 24><<<nb, kBlock, 0, s>>>(c->g, p0, np, lay, half, (const V *)native, (const V *)native + pv, (U *)user);
    HIP_CHECK(hipGetLastError());
}

template <typename S>
void spinor_io_user(dirac_ctx *c, void *native, const void *user, bool in, int sites, dirac_prec pr,
                    dirac_layout lay, hipStream_t s) {
    if (pr == DIRAC_F32)
        spinor_io<float, S>(c, native, user, in, sites, lay, s);
    else
        spinor_io<double, S>(c, native, user, in, sites, lay, s);
}

void spinor_dispatch(dirac_ctx *c, void *native, const void *user, bool in, int sites, dirac_prec pr,
                     dirac_layout lay, hipStream_t s) {
    require(lay == DIRAC_LAYOUT_LEX || lay == DIRAC_LAYOUT_EO || lay == DIRAC_LAYOUT_OPENQXD,
            "user layout must be LEX, EO or OPENQXD");
    require(sites >= 0 && sites <= 2, "sites must be 0 (full), 1 (even half) or 2 (odd half)");
    require(sites == 0 || lay != DIRAC_LAYOUT_LEX, "half vectors exist in the EO and OPENQXD layouts only");
    switch (pr) {
        case DIRAC_F64: spinor_io_user<double>(c, native, user, in, sites, pr, lay, s); break;
        case DIRAC_F32: spinor_io_user<float>(c, native, user, in, sites, pr, lay, s); break;
        case DIRAC_F16: spinor_io_user<__half>(c, native, user, in, sites, pr, lay, s); break;
        case DIRAC_BF16: spinor_io_user<__hip_bfloat16>(c, native, user, in, sites, pr, lay, s); break;
        default: throw Error(DIRAC_EINVAL, "unknown precision");
    }
}

// openQxD's gauge storage -> LEX: the thread of odd site (1, i) with ipt position V/2 + k reads the
// 8 links attached to it, slot 2 mu = U_mu(x) and slot 2 mu + 1 = U_mu(x - mu); every LEX link is
// written by exactly one thread (the forward link of an even site y ends at the odd site y + mu)
__global__ __launch_bounds__(kBlock) void k_openqxd_links(Geom g, const double *__restrict__ u_odd,
                                                           const double *__restrict__ a_odd,
                                                           double *__restrict__ U, double *__restrict__ th) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.vh) return;
    int x[4];
    site_coords(g, i, 1, x);
    const int64_t k = ipt_index(g, x) - g.vh;
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
#pragma unroll 1
        for (int back = 0; back < 2; ++back) {
            int y[4] = {x[0], x[1], x[2], x[3]};
            if (back) {
                const bool cross = y[mu] == 0;
                y[mu] = wrap_dn(y[mu], g.L[mu]);
                y[1] = cstar_x1(g, mu, cross, y[1]);  // C*: the link behind x may sit in the mirror copy
            }
            const int64_t lam = lex_index(g, y);
            const int64_t slot = k * 8 + 2 * mu + back;
            const double2 *src = reinterpret_cast<const double2 *>(u_odd) + slot * 9;
            double2 *dst = reinterpret_cast<double2 *>(U) + (lam * 4 + mu) * 9;
#pragma unroll
            for (int e = 0; e < 9; ++e) dst[e] = src[e];
            if (th) th[lam * 4 + mu] = a_odd[slot];
        }
    }
}

__global__ void k_zero16(size_t n, uint4 *__restrict__ p) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = make_uint4(0u, 0u, 0u, 0u);
}

}  // namespace

void zero_fill(void *p, size_t bytes, hipStream_t s) {
    const size_t n = bytes / 16;
    k_zero16<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, (uint4 *)p);
    HIP_CHECK(hipGetLastError());
}

void openqxd_links_to_lex(const Geom &g, const double *u_odd, const double *a_odd, double *U, double *th,
                          hipStream_t s) {
    k_openqxd_links<<<grid_for(g.vh), kBlock, 0, s>>>(g, u_odd, a_odd, U, th);
    HIP_CHECK(hipGetLastError());
}

size_t link_plane_bytes(dirac_prec pr) { return pr == DIRAC_F64 ? 96 : pr == DIRAC_F32 ? 48 : 24; }

void links_to_planes(const dirac_ctx *c, const void *su3_links, const double *theta, void *planes, hipStream_t s) {
    k_link_planes<<<c->g.vhp / kSB, kBlock, 0, s>>>(c->g, (const double2 *)su3_links, theta, (double2 *)planes,
                                                    theta_planes(planes, c->g));
    HIP_CHECK(hipGetLastError());
}

void import_links(dirac_ctx *c, const void *planes, const double *theta, hipStream_t s) {
    PrecFields &f = c->f[DIRAC_F64];
    c->flags.alloc(256);
    unsigned long long *maxdev = (unsigned long long *)c->flags.p;
    HIP_CHECK(hipMemsetAsync(maxdev, 0, sizeof(unsigned long long), s));
    const double4 ph = make_double4(c->p.bc_phase[0], c->p.bc_phase[1], c->p.bc_phase[2], c->p.bc_phase[3]);
    for (int p = 0; p < 2; ++p) {
        f.links[p].alloc_field((size_t)8 * 6 * sizeof(double2) * c->g.vhp);
        f.omega[p].alloc_field((size_t)8 * sizeof(double) * c->g.vhp);
        k_import_links<<<grid_for(c->vh), kBlock, 0, s>>>(c->g, p, (const double2 *)planes, theta, c->p.qhat, ph,
                                                          (double2 *)f.links[p].p, (double *)f.omega[p].p, maxdev);
    }
    HIP_CHECK(hipGetLastError());
    unsigned long long h = 0;
    HIP_CHECK(hipMemcpyAsync(&h, maxdev, sizeof(h), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    double dev;
    memcpy(&dev, &h, sizeof(dev));
    require(dev < 1e-10, "su3_links are not SU(3) matrices (max |U U^dag - 1| + |det U - 1| = " +
                             std::to_string(dev) + "); the two-row link compression needs det U = 1");
    f.links_ready = true;
}

void ensure_prec(dirac_ctx *c, dirac_prec pr, hipStream_t s) {
    switch (pr) {
        case DIRAC_F64: return;
        case DIRAC_F32: convert_fields<float>(c, pr, s); return;
        case DIRAC_F16: convert_fields<__half>(c, pr, s); return;
        case DIRAC_BF16: convert_fields<__hip_bfloat16>(c, pr, s); return;
        default: throw Error(DIRAC_EINVAL, "unknown precision");
    }
}

void spinor_import(dirac_ctx *c, void *native, const void *user, int sites, dirac_prec pr, dirac_layout lay,
                   hipStream_t s) {
    spinor_dispatch(c, native, user, true, sites, pr, lay, s);
}

void spinor_export(dirac_ctx *c, void *user, const void *native, int sites, dirac_prec pr, dirac_layout lay,
                   hipStream_t s) {
    spinor_dispatch(c, const_cast<void *>(native), user, false, sites, pr, lay, s);
}

void clover_import(dirac_ctx *c, const double *user, dirac_layout lay, hipStream_t s) {
    require(lay == DIRAC_LAYOUT_LEX || lay == DIRAC_LAYOUT_EO || lay == DIRAC_LAYOUT_OPENQXD,
            "clover layout must be LEX, EO or OPENQXD");
    PrecFields &f = c->f[DIRAC_F64];
    for (int p = 0; p < 2; ++p) f.clov[p].alloc_field((size_t)72 * sizeof(double) * c->g.vhp);
    k_site_in<double, double, 72><<<c->g.vhp / kSB, kBlock, 0, s>>>(c->g, 0, 2, lay, 0, user, (double2 *)f.clov[0].p,
                                                                     (double2 *)f.clov[1].p);
    HIP_CHECK(hipGetLastError());
    c->sap_ready = false;
    for (int q = 0; q < 4; ++q) {
        c->f[q].clover_ready = (q == DIRAC_F64);
        c->f[q].inv_ready[0] = c->f[q].inv_ready[1] = false;
    }
}

void clover_export(dirac_ctx *c, double *user, int inverse, dirac_layout lay, hipStream_t s) {
    require(lay == DIRAC_LAYOUT_LEX || lay == DIRAC_LAYOUT_EO || lay == DIRAC_LAYOUT_OPENQXD,
            "clover layout must be LEX, EO or OPENQXD");
    PrecFields &f = c->f[DIRAC_F64];
    const double2 *src[2];
    for (int p = 0; p < 2; ++p)
        src[p] = inverse ? (f.inv_ready[p] ? (const double2 *)f.clinv[p].p : nullptr) : (const double2 *)f.clov[p].p;
    k_site_out<double, double, 72><<<c->g.vhp / kSB, kBlock, 0, s>>>(c->g, 0, 2, lay, 0, src[0], src[1], user);
    HIP_CHECK(hipGetLastError());
}

}  // namespace dl
