// Clover field on the device (paper Sec. 4.3 and the outlook's "generate the clover
// field on the GPU"): build A = (4 + m0) + C from the SU(3) and U(1) links in FP64,
// invert its 6x6 chirality blocks in FP64 registers, and apply A or A^-1.
#include <type_traits>

#include "dirac_ops.h"
#include "internal.h"

namespace dl {
namespace {

struct M3 {
    C<double> m[9];
};

// t = t b or, DAG, t b^dag, row by row: one row more than t and b in registers
template <bool DAG>
DEV void mul_right(M3 &t, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        C<double> r[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            auto B = [&](int k) { return DAG ? conj(b.m[3 * j + k]) : b.m[3 * k + j]; };
            r[j] = t.m[3 * i] * B(0);
            madd(r[j], t.m[3 * i + 1], B(1));
            madd(r[j], t.m[3 * i + 2], B(2));
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) t.m[3 * i + j] = r[j];
    }
}

// F'_{mu nu}(x) = c_sw (Q - Q^dag)/8 + c_qed qhat (q - q*)/8, Q / q the sum of the four
// plaquette leaves at x in the (mu, nu) plane from U / from exp(i theta).  F' is anti-Hermitian: out
// holds its 9 independent reals, Im F_00, Im F_11, Im F_22, then (re, im) of F_01, F_02, F_12.
//
// Leaf l walks the steps c = l, l + 1, .. (mod 4) of +mu, +nu, -mu, -nu round from x and back, the links multiplied from
// the right as they are met: a rolled loop of 16 links, which holds the sum, the product and one link.
DEV void plane_field(const Geom &g, int p, const double2 *__restrict__ U, const double *__restrict__ th, const int x[4],
                     const double2 (*star)[9][kSB], int lane, int mu, int nu, double csw, double cq, double out[9]) {
    const bool u1 = th && cq != 0.0;
    int y[4] = {x[0], x[1], x[2], x[3]};
    M3 q, t;
    double ang = 0.0, sines = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) q.m[k] = t.m[k] = mk(0.0, 0.0);
#pragma nounroll
    for (int n = 0; n < 16; ++n) {
        const int c = ((n >> 2) + n) & 3, d = c & 1 ? nu : mu;
        const bool back = c >= 2;
        // one step along d; one that crosses the boundary of a C* direction also moves x1
        int z[4];
        bool cross = false;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int zm = back ? wrap_dn(y[m], g.L[m]) : wrap_up(y[m], g.L[m]);
            cross = cross || (m == d && (back ? zm > y[m] : zm < y[m]));
            z[m] = m == d ? zm : y[m];
        }
        z[1] = cstar_x1(g, d, cross, z[1]);
        int at[4];  // the site the link starts from
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            at[m] = back ? z[m] : y[m];
            y[m] = z[m];
        }
        const int par = p ^ ((n + (back ? 1 : 0)) & 1), i = half_index(g, at), s = n & 3;
        M3 u;
        if (s == 0 || s == 3) {
            const int e = 2 * d + ((s == 0) == back);
#pragma unroll
            for (int k = 0; k < 9; ++k) u.m[k] = mk(star[e][k][lane].x, star[e][k][lane].y);
        } else {
            const double2 *q9 = site_ptr(U + (size_t)(4 * par + d) * 9 * g.vhp, (uint32_t)i, 9);
#pragma unroll
            for (int k = 0; k < 9; ++k) u.m[k] = mk(q9[k * kSB].x, q9[k * kSB].y);
        }
        if (u1) {
            const double a = th[(size_t)(4 * par + d) * g.vhp + i];
            ang += back ? -a : a;
        }
        if (s == 0) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) t.m[3 * i + j] = back ? conj(u.m[3 * j + i]) : u.m[3 * i + j];
        } else if (back) {
            mul_right<true>(t, u);
        } else {
            mul_right<false>(t, u);
        }
        if (s == 3) {
#pragma unroll
            for (int k = 0; k < 9; ++k) q.m[k] = q.m[k] + t.m[k];
            if (u1) {
                double sn, cs;
                sc(ang, sn, cs);
                sines += sn;
                ang = 0.0;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) out[a] = (csw * 0.125) * (q.m[4 * a].i - (-q.m[4 * a].i));
    int k = 3;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a + 1; b < 3; ++b) {
            const C<double> f = (csw * 0.125) * (q.m[3 * a + b] - conj(q.m[3 * b + a]));
            out[k] = f.r;
            out[k + 1] = f.i;
            k += 2;
        }
    if (u1) {
        const double im = cq * 0.25 * sines;  // (q - q*) / 8 = i Im(q) / 4
#pragma unroll
        for (int a = 0; a < 3; ++a) out[a] += im;
    }
}

// A(x) packed as [72] reals, block + then block -, for the sites of parity p.
// With sigma_0k = diag(s_k, -s_k), sigma_jk = -eps_jkl diag(s_l, s_l) (chiral basis) the
// term (i/4) sum sigma_{mu nu} F_{mu nu} is, per chirality block, [[G3, G1 - i G2], [G1 + i G2, -G3]]:
//   block +: G1 = (i/2)(F01 - F23), G2 = (i/2)(F02 + F13), G3 = (i/2)(F03 - F12)
//   block -: G1 = -(i/2)(F01 + F23), G2 = -(i/2)(F02 - F13), G3 = -(i/2)(F03 + F12)
// A work-group of twelve wavefronts takes two blocks of 64 sites, one plane (mu, nu) and block per wavefront; the
// eight links at a site, which its planes use 48 times, are staged in LDS (one work-group on a CU: three
// wavefronts on each SIMD; work-groups of six wavefronts, on 2 + 2 + 1 + 1 SIMDs, ran one at a time even where two
// fitted), the fields meet there afterwards, and wavefront w forms planes 3 w .. 3 w + 2 of block + and of
// block - of its sites.  Bound by issue and the latency of its chain of products (16 steps of about 190 VALU
// instructions; with unstaged links, reading all of them at the own site saved 19 %, leaving the products out
// 2 %), against 0.15 ms for the FP64 operations alone.  24^3 x 48, a parity: 515 -> 456 us; 64 x 32^3 1.51 -> 1.35 ms.
constexpr int kFReals = 9;
__global__ __launch_bounds__(768, 3) void k_clover_build(Geom g, int p, const double2 *__restrict__ U,
                                                         const double *__restrict__ th, double csw, double cq,
                                                         double diag, double2 *__restrict__ out) {
    __shared__ double2 stars[2][8][9][kSB];  // slot 2 mu + back: the link from x or into x; then the fields
    const int lane = threadIdx.x & (kSB - 1), w12 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int sub = w12 >= 6, w = w12 - 6 * sub;
    const int first = 2 * xcd_block((int)gridDim.x);
    if (first * kSB >= g.vh) return;  // the whole work-group
    double2 (*star)[9][kSB] = stars[sub];
    double (*fs)[kFReals][kSB] = reinterpret_cast<double (*)[kFReals][kSB]>(&star[0][0][0]);
    const int blk = first + sub;
    const int i = min(blk * kSB + lane, g.vh - 1);  // lanes past the end repeat the last site
    int x[4];
    site_coords(g, i, p, x);
    {
        // the 72 planes of the star, 12 a wavefront: of slots e0 and e0 + 1
        const int e0 = 12 * w / 9, n0 = 9 * (e0 + 1) - 12 * w;
        const double2 *src[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int e = e0 + j, mu = e >> 1, back = e & 1;
            int y[4];
            bool cross = false;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int ym = back ? wrap_dn(x[m], g.L[m]) : x[m];
                cross = cross || (m == mu && ym > x[m]);
                y[m] = m == mu ? ym : x[m];
            }
            y[1] = cstar_x1(g, mu, cross, y[1]);
            src[j] = site_ptr(U + (size_t)(4 * (p ^ back) + mu) * 9 * g.vhp, (uint32_t)half_index(g, y), 9);
        }
        double2 v[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = k < n0 ? src[0][(9 - n0 + k) * kSB] : src[1][(k - n0) * kSB];
#pragma unroll
        for (int k = 0; k < 12; ++k) star[e0][0][(9 - n0 + k) * kSB + lane] = v[k];
        __syncthreads();
    }
    const int mu = w < 3 ? 0 : w < 5 ? 1 : 2, nu = w < 3 ? w + 1 : w < 5 ? w - 1 : 3;  // 01 02 03 12 13 23
    double f[kFReals];
    plane_field(g, p, U, th, x, star, lane, mu, nu, csw, cq, f);
    __syncthreads();  // the star is read before the fields take its place
#pragma unroll
    for (int k = 0; k < kFReals; ++k) fs[w][k][lane] = f[k];
    __syncthreads();
    if (blk * kSB + lane >= g.vh) return;  // no barrier follows
    // element k = 3 a + b of the anti-Hermitian field of plane n
    auto F = [&](int n, int k) -> C<double> {
        const int a = k / 3, b = k % 3;
        if (a == b) return mk(0.0, fs[n][a][lane]);
        const int lo = a < b ? a : b, hi = a < b ? b : a;
        const int q = 3 + 2 * (lo + hi - 1);
        const double re = fs[n][q][lane], im = fs[n][q + 1][lane];
        return a < b ? mk(re, im) : mk(-re, im);
    };
    double2 *dst = site_ptr(out, (uint32_t)i, 36);
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        // G1, G2, G3 of the block: block + (F01 - F23, F02 + F13, F03 - F12) * (i/2), block -
        // -(F01 + F23, F02 - F13, F03 + F12) * (i/2)
        auto G1 = [&](int k) { return 0.5 * times_i(blk == 0 ? F(0, k) - F(5, k) : -(F(0, k) + F(5, k))); };
        auto G2 = [&](int k) { return 0.5 * times_i(blk == 0 ? F(1, k) + F(4, k) : -(F(1, k) - F(4, k))); };
        auto G3 = [&](int k) { return 0.5 * times_i(blk == 0 ? F(2, k) - F(3, k) : -(F(2, k) + F(3, k))); };
        auto B = [&](int r, int c) -> C<double> {
            const int s = r / 3, t = c / 3, k = 3 * (r % 3) + c % 3;
            C<double> v;
            if (s == 0 && t == 0) v = G3(k);
            else if (s == 0 && t == 1) v = G1(k) - times_i(G2(k));
            else if (s == 1 && t == 0) v = G1(k) + times_i(G2(k));
            else v = -G3(k);
            if (r == c) v.r += diag;
            return v;
        };
        // packed plane j: the diagonal in pairs for j < 3, then one strictly-upper entry each
        auto plane = [&](int j) {
            if (j < 3) return make_double2(B(2 * j, 2 * j).r, B(2 * j + 1, 2 * j + 1).r);
            int r = 0, c = j - 2;  // entry j - 3 of the upper triangle, row-major
            while (c > 5) {
                ++r;
                c = c - 5 + r;
            }
            const C<double> v = B(r, c);
            return make_double2(v.r, v.i);
        };
        auto put = [&](auto first) {
            constexpr int J = decltype(first)::value;
            dst[(18 * blk + J) * kSB] = plane(J);
            dst[(18 * blk + J + 1) * kSB] = plane(J + 1);
            dst[(18 * blk + J + 2) * kSB] = plane(J + 2);
        };
        switch (w) {
            case 0: put(std::integral_constant<int, 0>()); break;
            case 1: put(std::integral_constant<int, 3>()); break;
            case 2: put(std::integral_constant<int, 6>()); break;
            case 3: put(std::integral_constant<int, 9>()); break;
            case 4: put(std::integral_constant<int, 12>()); break;
            default: put(std::integral_constant<int, 15>()); break;
        }
    }
}

// Gauss-Jordan inversion of a 6x6 complex block with partial pivoting (pivot row chosen by
// max |re| + |im| as in LAPACK's zgetrf).  Returns false when a pivot modulus is below thr.
DEV bool invert6(C<double> a[6][6], C<double> v[6][6], double thr) {
    bool ok = true;
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c) v[r][c] = mk(r == c ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        int piv = k;
        double best = fabs(a[k][k].r) + fabs(a[k][k].i);
#pragma unroll
        for (int r = k + 1; r < 6; ++r) {
            double m = fabs(a[r][k].r) + fabs(a[r][k].i);
            if (m > best) { best = m; piv = r; }
        }
#pragma unroll
        for (int r = k + 1; r < 6; ++r) {
            const bool sw = (piv == r);
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                C<double> t = a[k][c], u = a[r][c];
                a[k][c] = sw ? u : t;
                a[r][c] = sw ? t : u;
                t = v[k][c]; u = v[r][c];
                v[k][c] = sw ? u : t;
                v[r][c] = sw ? t : u;
            }
        }
        const C<double> pv = a[k][k];
        const double n2 = pv.r * pv.r + pv.i * pv.i;
        if (!(sqrt(n2) >= thr)) ok = false;
        const double inv = n2 > 0.0 ? 1.0 / n2 : 0.0;
        const C<double> rp = mk(pv.r * inv, -pv.i * inv);  // 1 / pivot
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            a[k][c] = a[k][c] * rp;
            v[k][c] = v[k][c] * rp;
        }
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            if (r == k) continue;
            const C<double> f = a[r][k];
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                a[r][c] = a[r][c] - f * a[k][c];
                v[r][c] = v[r][c] - f * v[k][c];
            }
        }
    }
    return ok;
}

__global__ __launch_bounds__(kBlock) void k_clover_invert(Geom g, int p, const double2 *__restrict__ A,
                                                           double2 *__restrict__ Ainv, int *__restrict__ first_bad) {
    int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.vh) return;
    bool ok = true;
    double out[72];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        double pk[36];
        const double2 *Ai = site_ptr(A, (uint32_t)i, 36);
#pragma unroll
        for (int k = 0; k < 18; ++k) {
            double2 v = Ai[(18 * blk + k) * kSB];
            pk[2 * k] = v.x;
            pk[2 * k + 1] = v.y;
        }
        C<double> a[6][6], v[6][6];
        double amax = 0.0;
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            a[r][r] = mk(pk[r], 0.0);
            amax = fmax(amax, fabs(pk[r]));
        }
        int k = 6;
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r + 1; c < 6; ++c) {
                a[r][c] = mk(pk[k], pk[k + 1]);
                a[c][r] = mk(pk[k], -pk[k + 1]);
                amax = fmax(amax, sqrt(pk[k] * pk[k] + pk[k + 1] * pk[k + 1]));
                k += 2;
            }
        ok = invert6(a, v, 1e-14 * amax) && ok;
        double *o = out + 36 * blk;
#pragma unroll
        for (int r = 0; r < 6; ++r) o[r] = v[r][r].r;
        k = 6;
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r + 1; c < 6; ++c) {
                o[k] = v[r][c].r;
                o[k + 1] = v[r][c].i;
                k += 2;
            }
    }
    store_field<double, 72>(Ainv, (uint32_t)i, out);
    if (!ok) {
        int x[4];
        site_coords(g, i, p, x);
        atomicMin(first_bad, lex_index(g, x));
    }
}

template <typename S, int INV>
__global__ __launch_bounds__(kBlock) void k_clover_apply(int vh, size_t vs, const typename St<S>::vec *__restrict__ in,
                                                          const typename St<S>::vec *__restrict__ A,
                                                          typename St<S>::vec *__restrict__ out) {
    using T = typename St<S>::acc;
    int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= vh) return;
    in += blockIdx.y * vs;  // right-hand side blockIdx.y
    out += blockIdx.y * vs;
    T r[24], pk[72];
    load_field<S, 24>(in, (uint32_t)i, r);
    load_field<S, 72>(A, (uint32_t)i, pk);
    C<T> psi[12], y[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) psi[k] = mk(r[2 * k], r[2 * k + 1]);
    block_mul(pk, psi, y);
    block_mul(pk + 36, psi + 6, y + 6);
#pragma unroll
    for (int k = 0; k < 12; ++k) { r[2 * k] = y[k].r; r[2 * k + 1] = y[k].i; }
    store_field<S, 24>(out, (uint32_t)i, r);
}

template <typename S>
void clover_apply_t(dirac_ctx *c, void *out, const void *in, int parity, int inverse, dirac_prec pr, hipStream_t s,
                    int nrhs) {
    PrecFields &f = c->f[pr];
    const void *A = inverse ? f.clinv[parity].p : f.clov[parity].p;
    using V = typename St<S>::vec;
    const size_t vs = (size_t)(24 / St<S>::W) * c->g.vhp;
    const dim3 grid(grid_for(c->vh), nrhs);
    if (inverse)
        k_clover_apply<S, 1><<<grid, kBlock, 0, s>>>((int)c->vh, vs, (const V *)in, (const V *)A, (V *)out);
    else
        k_clover_apply<S, 0><<<grid, kBlock, 0, s>>>((int)c->vh, vs, (const V *)in, (const V *)A, (V *)out);
    HIP_CHECK(hipGetLastError());
}

}  // namespace

void clover_build(dirac_ctx *c, const void *planes, const double *theta, hipStream_t s) {
    PrecFields &f = c->f[DIRAC_F64];
    const double diag = 1.0 / (2.0 * c->p.kappa);
    for (int p = 0; p < 2; ++p) {
        f.clov[p].alloc_field((size_t)72 * sizeof(double) * c->g.vhp);
        k_clover_build<<<((c->g.vhp / kSB + 1) / 2 + 7) & ~7, 768, 0, s>>>(c->g, p, (const double2 *)planes, theta, c->p.csw,
                                                      c->p.csw_qed * c->p.qhat, diag, (double2 *)f.clov[p].p);
    }
    HIP_CHECK(hipGetLastError());
    c->sap_ready = false;
    for (int q = 0; q < 4; ++q) {
        c->f[q].clover_ready = (q == DIRAC_F64);
        c->f[q].inv_ready[0] = c->f[q].inv_ready[1] = false;
    }
}

int64_t clover_invert_parity(dirac_ctx *c, int p, hipStream_t s) {
    PrecFields &f = c->f[DIRAC_F64];
    require(f.clover_ready, "no clover field");
    f.clinv[p].alloc_field((size_t)72 * sizeof(double) * c->g.vhp);
    c->flags.alloc(256);
    int *bad = (int *)c->flags.p + 8;
    const int big = 0x7fffffff;
    HIP_CHECK(hipMemcpyAsync(bad, &big, sizeof(int), hipMemcpyHostToDevice, s));
    k_clover_invert<<<grid_for(c->vh), kBlock, 0, s>>>(c->g, p, (const double2 *)f.clov[p].p,
                                                       (double2 *)f.clinv[p].p, bad);
    HIP_CHECK(hipGetLastError());
    int h = big;
    HIP_CHECK(hipMemcpyAsync(&h, bad, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    for (int q = 0; q < 4; ++q) c->f[q].inv_ready[p] = false;
    f.inv_ready[p] = true;
    return h == big ? -1 : (int64_t)h;
}

void clover_apply(dirac_ctx *c, void *out, const void *in, int parity, int inverse, dirac_prec pr, hipStream_t s,
                  int nrhs) {
    require(parity == 0 || parity == 1, "parity must be 0 (even) or 1 (odd)");
    ensure_prec(c, pr, s);
    PrecFields &f = c->f[pr];
    require(!inverse || f.inv_ready[parity], "clover inverse of this parity not computed; call clover_invert");
    switch (pr) {
        case DIRAC_F64: clover_apply_t<double>(c, out, in, parity, inverse, pr, s, nrhs); break;
        case DIRAC_F32: clover_apply_t<float>(c, out, in, parity, inverse, pr, s, nrhs); break;
        case DIRAC_F16: clover_apply_t<__half>(c, out, in, parity, inverse, pr, s, nrhs); break;
        case DIRAC_BF16: clover_apply_t<__hip_bfloat16>(c, out, in, parity, inverse, pr, s, nrhs); break;
        default: throw Error(DIRAC_EINVAL, "unknown precision");
    }
}

}  // namespace dl
