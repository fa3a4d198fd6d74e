// Schwarz alternating procedure (SAP): the block preconditioner of openQxD's solver, on 4^4
// blocks coloured as a checkerboard of blocks.  One application psi = M r:
//   psi = 0, rho = r; ncy times, for colour 0 then colour 1: on every block of the colour,
//   delta = nmr minimal-residual steps on the block operator D_blk (hops that leave the block
//   dropped) for the residual on the block; psi += delta; rho = r - D psi.
// One work-group per block, one thread per site.  The residual of the block is staged in LDS
// (the neighbour reads of D_blk), and so are the block's links of in-block hops and, in
// registers, each site's clover block: they are read from memory once per block solve, not once
// per minimal-residual step.  The block reductions of the minimal-residual steps are
// shuffle trees and a fixed-order sum over the four wavefronts (deterministic).  The residual
// update after a colour's solves changes rho only on the faces of the other colour's blocks
// (D delta = -1/2 H delta there); it is done by the next step's work-groups on entry, from the
// corrections delta of the previous step, kept projected on the faces, so a step is one launch.  FP32 throughout (the
// arithmetic of a preconditioner), on block-ordered copies of the F32 links and clover field.
#include "dirac_ops.h"
#include "hop_core.h"
#include "internal.h"

namespace dl {
namespace {

constexpr int kSapB = 4;                                  // block extent in every direction
constexpr int kSapSites = kSapB * kSapB * kSapB * kSapB;  // 256: one work-group
constexpr int kSapInner = kSapSites / kSapB * (kSapB - 1);  // 192 sites of a block with a neighbour inside it in +mu
constexpr int kSapFace = kSapSites / kSapB;                 // 64 sites of a face
// Links of a block: the 4 x 192 of hops inside it, then the 8 x 64 of hops into it across its faces; of each
// list three planes (rows 0 and 1 of the SU(3) matrix), then (cos, sin) of the phase; in float4:
constexpr int kSapInnerPh = 4 * 3 * kSapInner, kSapFaces = kSapInnerPh + 4 * kSapInner / 2;
constexpr int kSapFacePh = kSapFaces + 8 * 3 * kSapFace, kSapLinks = kSapFacePh + 8 * kSapFace / 2;

// Block order: the fields of the Schwarz blocks are kept block by block (block k lexicographic in
// the block coordinates, site t = 64 b0 + 16 b1 + 4 b2 + b3 inside it), plane-major within a
// block, so that a work-group reads one contiguous chunk and every wavefront load is 1 KB of
// consecutive 16-byte vectors:  spinor [k][6][256], clover [k][18][256], links as above, 70 KB a block, and
// the corrections on the faces [k][8][3][64].
// (The sites of a 4^4 block lie in 2-site pieces of the x3-fastest NATIVE order: read from there,
// every wavefront load touches 32 cache lines for 32 bytes each.  The first cycle reads the
// residual from there all the same, which costs less than a separate reordering pass; the
// solution goes back through one, as scattered 32-byte writes of partial cache lines from the
// last cycle's steps cost more than the pass.)
struct SapArgs {
    Geom g;
    const float4 *links;  // block order
    const float4 *clov;   // block order
    float4 *rho, *psi;    // block order, all blocks
    float4 *faces;        // block k, direction d: delta on the face that is the source of its neighbour's hops d, projected
    const float4 *rin;    // NATIVE input residual, read instead of rho when set (the first cycle)
    int nb[4];            // blocks per direction
    int colour, nmr, update;
    int first;            // the first cycle: psi is zero, so psi = delta
    int keep;             // rho is read again (not in the last cycle)
    int send;             // the faces are read by a further step
};

DEV int block_of(const SapArgs &a, const int n[4]) { return ((n[0] * a.nb[1] + n[1]) * a.nb[2] + n[2]) * a.nb[3] + n[3]; }
DEV size_t spinor_at(int k, int t) { return (size_t)k * 6 * kSapSites + t; }  // plane 0; plane j at + j * 256

// Block coordinates of the k-th block of colour c: blocks are lexicographic in (n0, n1, n2, n3),
// and every row of n3 (an even number of blocks) holds half of each colour.
DEV void sap_block(const SapArgs &a, int k, int n[4]) {
    const int half3 = a.nb[3] / 2;
    const int r = k / half3, m = k % half3;
    n[2] = r % a.nb[2];
    n[1] = (r / a.nb[2]) % a.nb[1];
    n[0] = r / (a.nb[2] * a.nb[1]);
    n[3] = 2 * m + ((a.colour + n[0] + n[1] + n[2]) & 1);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

DEV void load_sp(const float4 *base, C<float> r[12]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float4 q = base[k * kSapSites];
        r[2 * k] = mk(q.x, q.y);
        r[2 * k + 1] = mk(q.z, q.w);
    }
}
DEV void store_sp(float4 *base, const C<float> r[12]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) base[k * kSapSites] = make_float4(r[2 * k].r, r[2 * k].i, r[2 * k + 1].r, r[2 * k + 1].i);
}
// Forward link of direction mu at block site t (b_mu < 3, the links of the hops inside the block),
// in the LDS tile of the block: the 192 such sites of a direction, in site order.
DEV int inner_link(int mu, int t) {
    const int sh = 6 - 2 * mu;  // log2 of the site stride of direction mu
    return t - ((t >> (sh + 2)) << sh);
}

// The other three coordinates of a block site, x3 fastest: its place on a face of direction mu.
DEV int face_site(int mu, const int b[4]) {
    int f = 0, o = 0;
#pragma unroll
    for (int m = 3; m >= 0; --m) {
        if (m == mu) continue;
        f |= b[m] << (2 * o);
        ++o;
    }
    return f;
}

template <int N = 0, typename F>
DEV void each_dir(const F &f) {
    f(std::integral_constant<int, N>());
    if constexpr (N < 7) each_dir<N + 1>(f);
}

DEV void cplx3(float4 p, float4 q, float4 r, C<float> o[6]) {
    o[0] = mk(p.x, p.y); o[1] = mk(p.z, p.w);
    o[2] = mk(q.x, q.y); o[3] = mk(q.z, q.w);
    o[4] = mk(r.x, r.y); o[5] = mk(r.z, r.w);
}
DEV float4 pair4(C<float> p, C<float> q) { return make_float4(p.r, p.i, q.r, q.i); }

// w = M h (forward) or M^dag h (backward) for both spin rows; M, the link times its phase, in full.
template <int BACK>
DEV void full_mul(const C<float> M[9], const C<float> h[6], C<float> w[6]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            C<float> t = BACK ? conj_mul(M[r], h[3 * s]) : M[3 * r] * h[3 * s];
#pragma unroll
            for (int c = 1; c < 3; ++c) {
                if constexpr (BACK) cmadd(t, M[3 * c + r], h[3 * s + c]);
                else madd(t, M[3 * r + c], h[3 * s + c]);
            }
            w[3 * s + r] = t;
        }
}

// One step: the face terms of the other colour's last corrections, nmr minimal-residual steps, the results.
// At 4 minimal-residual steps it moves 1.1 KB a site (0.85 KB of it read) and issues 6,600 VALU instructions a
// wavefront, and two work-groups fit on a CU (80 KB of LDS and 239 registers each), which overlap only in part.  So
//  - the block's inner links are kept in LDS as full matrices with their phase: third row and phase
//    product are formed once a step, not in each of the 4 x 7.5 hops of a site (8,150 instructions before);
//  - only the projected faces of the corrections travel between blocks, 48 of 96 bytes a site, in whole
//    cache lines (a face of direction 3 is every fourth site of the block), and only the links that are
//    used (1.36 GB read a step before on 64 x 32^3, 0.92 GB now);
//  - all loads of the entry are issued together, before the first is waited for.
// On 64 x 32^3 with 4 cycles of 4 steps: 343 -> 276 us a step, 71 % of the SIMD cycles issue VALU instructions.
// -1/2 folded into the links, hops added to A r directly: 272 us, but the rounding error grows by 5 %.
__global__ __launch_bounds__(kSapSites) void k_sap_step(SapArgs a) {
    // the face terms [8][3][64], then the block's residual [6][256]
    __shared__ float4 rs[6 * kSapSites];
    __shared__ float red[3][4];
    // links of the hops inside the block, phase included (a backward hop from t takes the forward link of
    // t - stride): 18 reals as four planes of float4 and one of float2
    __shared__ float4 lq[4][4][kSapInner];
    __shared__ float2 lr[4][kSapInner];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int b[4] = {t >> 6, (t >> 4) & 3, (t >> 2) & 3, t & 3};
    int n[4];
    sap_block(a, blockIdx.x, n);
    const int k = block_of(a, n);
    const float4 *lk = a.links + (size_t)k * kSapLinks;

    // face terms: wavefront w takes the faces of directions w and w + 4, a lane a site
    float4 fh[2][3], fu[2][3];
    float2 fp[2];
    if (a.update) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int d = 4 * j + wave, mu = d >> 1, back = d & 1;
            // the neighbouring block, with the lattice wrap and the C* mirror shift
            int nn[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) nn[m] = n[m];
            const int nm = mu == 0 ? n[0] : mu == 1 ? n[1] : mu == 2 ? n[2] : n[3];
            const int Nm = mu == 0 ? a.nb[0] : mu == 1 ? a.nb[1] : mu == 2 ? a.nb[2] : a.nb[3];
            const bool cross = back ? nm == 0 : nm == Nm - 1;
            const int nx = back ? (cross ? Nm - 1 : nm - 1) : (cross ? 0 : nm + 1);
            if (mu == 0) nn[0] = nx; else if (mu == 1) nn[1] = nx; else if (mu == 2) nn[2] = nx; else nn[3] = nx;
            nn[1] = cstar_x1(a.g, mu, cross, kSapB * nn[1]) / kSapB;
            const float4 *src = a.faces + ((size_t)block_of(a, nn) * 8 + d) * 3 * kSapFace + lane;
            const float4 *ul = lk + kSapFaces + d * 3 * kSapFace + lane;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                fh[j][q] = src[q * kSapFace];
                fu[j][q] = ul[q * kSapFace];
            }
            fp[j] = reinterpret_cast<const float2 *>(lk + kSapFacePh)[d * kSapFace + lane];
        }
    }
    float4 iu[3][3];
    float2 ip[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int e = t + j * kSapSites, mu = e / kSapInner, ci = e % kSapInner;
#pragma unroll
        for (int q = 0; q < 3; ++q) iu[j][q] = lk[(mu * 3 + q) * kSapInner + ci];
        ip[j] = reinterpret_cast<const float2 *>(lk + kSapInnerPh)[e];
    }
    C<float> r[12];
    if (a.rin) {
        // the site's position in the NATIVE full vectors (parity-major, 6 planes per site)
        int xs[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) xs[m] = kSapB * n[m] + b[m];
        const int par = (xs[0] + xs[1] + xs[2] + xs[3]) & 1;
        const int hi = half_index(a.g, xs);
        const size_t nat = (size_t)par * 6 * a.g.vhp + (size_t)(hi >> 6) * 6 * kSB + (hi & (kSB - 1));
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const float4 v = a.rin[nat + q * kSB];
            r[2 * q] = mk(v.x, v.y);
            r[2 * q + 1] = mk(v.z, v.w);
        }
    } else {
        load_sp(a.rho + spinor_at(k, t), r);
    }
    // the site's clover block, read once for all minimal-residual steps
    float pk[72];
    {
        const float4 *cq = a.clov + (size_t)k * 18 * kSapSites + t;
#pragma unroll
        for (int q = 0; q < 18; ++q) {
            const float4 f = cq[q * kSapSites];
            pk[4 * q] = f.x;
            pk[4 * q + 1] = f.y;
            pk[4 * q + 2] = f.z;
            pk[4 * q + 3] = f.w;
        }
    }

    if (a.update) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int d = 4 * j + wave;
            C<float> h[6], u[6], w[6];
            cplx3(fh[j][0], fh[j][1], fh[j][2], h);
            cplx3(fu[j][0], fu[j][1], fu[j][2], u);
            if (d & 1) link_adj_mul(u, fp[j].x, fp[j].y, h, w);
            else link_mul(u, fp[j].x, fp[j].y, h, w);
            float4 *dst = rs + d * 3 * kSapFace + lane;
#pragma unroll
            for (int q = 0; q < 3; ++q) dst[q * kSapFace] = pair4(w[2 * q], w[2 * q + 1]);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int e = t + j * kSapSites, mu = e / kSapInner, ci = e % kSapInner;
        C<float> u[6], M[9];
        cplx3(iu[j][0], iu[j][1], iu[j][2], u);
        third_row(u, M + 6);
        const C<float> ph = mk(ip[j].x, ip[j].y);
#pragma unroll
        for (int q = 0; q < 9; ++q) M[q] = ph * (q < 6 ? u[q < 6 ? q : 0] : M[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) lq[mu][q][ci] = pair4(M[2 * q], M[2 * q + 1]);
        lr[mu][ci] = make_float2(M[8].r, M[8].i);
    }
    if (a.update) {
        // rho += 1/2 H delta: a site adds the terms of the faces it is on, in direction order
        __syncthreads();
        C<float> acc[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) acc[q] = mk(0.f, 0.f);
        each_dir([&](auto dn) {
            constexpr int N = dn, mu = N >> 1, back = N & 1;
            if (b[mu] != (back ? 0 : kSapB - 1)) return;  // not on this face
            const float4 *src = rs + N * 3 * kSapFace + face_site(mu, b);
            C<float> w[6];
            cplx3(src[0], src[kSapFace], src[2 * kSapFace], w);
            add_rows_n<float, 0, N>(w, acc);
        });
#pragma unroll
        for (int q = 0; q < 12; ++q) r[q] = mk(fmaf(0.5f, acc[q].r, r[q].r), fmaf(0.5f, acc[q].i, r[q].i));
        __syncthreads();  // the terms are read before the residual takes their place
    }
    C<float> dl_[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) dl_[q] = mk(0.f, 0.f);

    // Two barriers a step: the second orders this step's reads of rs before the next step's writes, the first the
    // reads of red before the next writes of it (and the links before their first use).
#pragma nounroll
    for (int it = 0; it < a.nmr; ++it) {
#pragma unroll
        for (int q = 0; q < 6; ++q) rs[q * kSapSites + t] = pair4(r[2 * q], r[2 * q + 1]);
        __syncthreads();
        // v = D_blk r = A r - 1/2 sum over the neighbours inside the block
        C<float> v[12], hs[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) hs[q] = mk(0.f, 0.f);
        each_dir([&](auto dn) {
            constexpr int N = dn, mu = N >> 1, back = N & 1;
            constexpr int stride = mu == 0 ? 64 : mu == 1 ? 16 : mu == 2 ? 4 : 1;
            if (b[mu] == (back ? 0 : kSapB - 1)) return;  // that neighbour is outside the block
            const int tn = back ? t - stride : t + stride;
            C<float> nb[12], h[6], M[9], w[6];
            cplx3(rs[tn], rs[kSapSites + tn], rs[2 * kSapSites + tn], nb);
            cplx3(rs[3 * kSapSites + tn], rs[4 * kSapSites + tn], rs[5 * kSapSites + tn], nb + 6);
            const int ci = inner_link(mu, back ? tn : t);
            cplx3(lq[mu][0][ci], lq[mu][1][ci], lq[mu][2][ci], M);
            const float4 l3 = lq[mu][3][ci];
            const float2 l4 = lr[mu][ci];
            M[6] = mk(l3.x, l3.y); M[7] = mk(l3.z, l3.w); M[8] = mk(l4.x, l4.y);
            project_dir_n<float, 0, N>(nb, h);
            full_mul<back>(M, h, w);
            add_rows_n<float, 0, N>(w, hs);
        });
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) block_mul(pk + 36 * blk, r + 6 * blk, v + 6 * blk);
#pragma unroll
        for (int q = 0; q < 12; ++q) v[q] = mk(fmaf(-0.5f, hs[q].r, v[q].r), fmaf(-0.5f, hs[q].i, v[q].i));
        // w = <v, r> / <v, v> over the block
        float vr = 0.f, vi = 0.f, vv = 0.f;
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            vr = fmaf(v[q].r, r[q].r, fmaf(v[q].i, r[q].i, vr));
            vi = fmaf(v[q].r, r[q].i, fmaf(-v[q].i, r[q].r, vi));
            vv = fmaf(v[q].r, v[q].r, fmaf(v[q].i, v[q].i, vv));
        }
        vr = wave_sum(vr);
        vi = wave_sum(vi);
        vv = wave_sum(vv);
        if (lane == 0) {
            red[0][wave] = vr;
            red[1][wave] = vi;
            red[2][wave] = vv;
        }
        __syncthreads();
        const float sr = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        const float si = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
        const float sv = (red[2][0] + red[2][1]) + (red[2][2] + red[2][3]);
        const float inv = sv > 0.f ? 1.0f / sv : 0.f;
        const C<float> w = mk(sr * inv, si * inv);
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            madd(dl_[q], w, r[q]);
            madd(r[q], mk(-w.r, -w.i), v[q]);
        }
    }
    // psi += delta, rho = the block residual, the faces of delta for the next step's update
    float4 *ps = a.psi + spinor_at(k, t);
    C<float> o[12];
    if (a.first) {
#pragma unroll
        for (int q = 0; q < 12; ++q) o[q] = dl_[q];
    } else {
        load_sp(ps, o);
#pragma unroll
        for (int q = 0; q < 12; ++q) o[q] = mk(o[q].r + dl_[q].r, o[q].i + dl_[q].i);
    }
    store_sp(ps, o);
    if (a.keep) store_sp(a.rho + spinor_at(k, t), r);
    if (!a.send) return;
    each_dir([&](auto dn) {
        constexpr int N = dn, mu = N >> 1, back = N & 1;
        if (b[mu] != (back ? kSapB - 1 : 0)) return;  // the neighbour's hop N does not start here
        C<float> h[6];
        project_dir_n<float, 0, N>(dl_, h);
        float4 *dst = a.faces + ((size_t)k * 8 + N) * 3 * kSapFace + face_site(mu, b);
#pragma unroll
        for (int q = 0; q < 3; ++q) dst[q * kSapFace] = pair4(h[2 * q], h[2 * q + 1]);
    });
}

// Block order of the fields (once per field): site (p, i) -> block k, site t
DEV void block_pos(const Geom &g, const int nb[4], const int x[4], int &k, int &t) {
    int n[4], b[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        n[m] = x[m] / kSapB;
        b[m] = x[m] % kSapB;
    }
    k = ((n[0] * nb[1] + n[1]) * nb[2] + n[2]) * nb[3] + n[3];
    t = ((b[0] * kSapB + b[1]) * kSapB + b[2]) * kSapB + b[3];
}

// Both sites of a pair per thread, as in k_sap_unorder: the two parities' pieces of a cache line are written together
// (2 x 0.72 -> 0.78 ms on 64 x 32^3, once per field).
struct SapFields {
    const float4 *links, *clov;
    const float *omega;
};
__global__ void k_sap_fields(Geom g, int4 nb4, SapFields even, SapFields odd, float4 *__restrict__ blinks,
                             float4 *__restrict__ bclov) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.vh) return;
    const int nb[4] = {nb4.x, nb4.y, nb4.z, nb4.w};
    const size_t vhp = (size_t)g.vhp;
    int k[2], t[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        int x[4];
        site_coords(g, i, p, x);
        block_pos(g, nb, x, k[p], t[p]);
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int mu = d >> 1;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const SapFields &f = p ? odd : even;
            const int b[4] = {t[p] >> 6, (t[p] >> 4) & 3, (t[p] >> 2) & 3, t[p] & 3};
            const bool face = b[mu] == (d & 1 ? 0 : kSapB - 1);
            if (!face && (d & 1)) continue;  // the forward link of t - stride serves this hop
            const int n = face ? kSapFace : kSapInner, at = face ? face_site(mu, b) : inner_link(mu, t[p]);
            const int list = face ? d : mu;
            const float4 *src = site_ptr(f.links + (size_t)d * 3 * vhp, (uint32_t)i, 3);
            float4 *lk = blinks + (size_t)k[p] * kSapLinks, *dst = lk + (face ? kSapFaces : 0) + list * 3 * n + at;
            dst[0] = src[0];
            dst[n] = src[kSB];
            dst[2 * n] = src[2 * kSB];
            float sn, cs;
            sc(f.omega[(size_t)d * vhp + i], sn, cs);
            reinterpret_cast<float2 *>(lk + (face ? kSapFacePh : kSapInnerPh))[list * n + at] = make_float2(cs, sn);
        }
    }
#pragma unroll
    for (int q = 0; q < 18; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            bclov[(size_t)k[p] * 18 * kSapSites + t[p] + q * kSapSites] =
                site_ptr((p ? odd : even).clov, (uint32_t)i, 18)[q * kSB];
}

// Block order -> NATIVE F32 full vector (the solution at the end of an application).  A thread takes both sites 2 i
// and 2 i + 1 of a row: the block's cache lines hold the two parities alternately, and a launch per parity read
// them twice (2 x 48 -> 68 us on 64 x 32^3, the rate of a copy).
__global__ void k_sap_unorder(Geom g, int4 nb4, float4 *__restrict__ nat, const float4 *__restrict__ blk) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.vh) return;
    const int nb[4] = {nb4.x, nb4.y, nb4.z, nb4.w};
    float4 v[2][6];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        int x[4], k, t;
        site_coords(g, i, p, x);
        block_pos(g, nb, x, k, t);
        const float4 *bq = blk + spinor_at(k, t);
#pragma unroll
        for (int j = 0; j < 6; ++j) v[p][j] = bq[j * kSapSites];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        float4 *q = site_ptr(nat + (size_t)p * 6 * g.vhp, (uint32_t)i, 6);
#pragma unroll
        for (int j = 0; j < 6; ++j) q[j * kSB] = v[p][j];
    }
}

}  // namespace

bool sap_supported(const dirac_ctx *c) {
    for (int m = 0; m < 4; ++m)
        if (c->g.L[m] % (2 * kSapB) != 0) return false;
    // C*: crossing a shifted boundary moves x1 by L1/2, which must be an even number of blocks,
    // or two blocks of one colour would meet across that face
    if (c->g.cs >= 2 && c->g.h1 % (2 * kSapB) != 0) return false;
    return true;
}

// psi = M_SAP r on NATIVE F32 full vectors
void sap_apply(dirac_ctx *c, void *psi, const void *r, int ncy, int nmr, hipStream_t s) {
    require(sap_supported(c), "the Schwarz preconditioner needs every lattice extent to be a multiple of 8 "
                              "(an even number of 4^4 blocks per direction) and, with C* boundaries, dims[1] a "
                              "multiple of 16");
    require(ncy >= 1 && ncy <= 64 && nmr >= 1 && nmr <= 64, "SAP cycles and block steps must be 1..64");
    ensure_prec(c, DIRAC_F32, s);
    int nblk = 1;
    int nb[4];
    for (int m = 0; m < 4; ++m) {
        nb[m] = c->g.L[m] / kSapB;
        nblk *= nb[m];
    }
    const int4 nb4 = make_int4(nb[0], nb[1], nb[2], nb[3]);
    const int vh = (int)c->vh;
    if (!c->sap_ready) {
        c->sap_links.alloc((size_t)nblk * kSapLinks * sizeof(float4));
        c->sap_clov.alloc((size_t)nblk * 18 * kSapSites * sizeof(float4));
        SapFields f[2];
        for (int p = 0; p < 2; ++p)
            f[p] = {(const float4 *)c->f[DIRAC_F32].links[p].p, (const float4 *)c->f[DIRAC_F32].clov[p].p,
                    (const float *)c->f[DIRAC_F32].omega[p].p};
        k_sap_fields<<<grid_for(vh), kBlock, 0, s>>>(c->g, nb4, f[0], f[1], (float4 *)c->sap_links.p, (float4 *)c->sap_clov.p);
        HIP_CHECK(hipGetLastError());
        c->sap_ready = true;
    }
    const size_t vbytes = (size_t)nblk * 6 * kSapSites * sizeof(float4);
    c->sap_rho.alloc(3 * vbytes);  // rho, psi, the faces (8 x 3 x 64 = 6 x 256) in block order
    float4 *rho = (float4 *)c->sap_rho.p, *pb = rho + vbytes / sizeof(float4), *faces = pb + vbytes / sizeof(float4);
    // the first cycle reads the residual from the NATIVE input (no reordering pass in), and psi
    // starts as the first cycle's corrections (no zero fill)
    SapArgs a{};
    a.g = c->g;
    a.links = (const float4 *)c->sap_links.p;
    a.clov = (const float4 *)c->sap_clov.p;
    a.rho = rho;
    a.psi = pb;
    a.faces = faces;
    for (int m = 0; m < 4; ++m) a.nb[m] = nb[m];
    a.nmr = nmr;
    for (int cy = 0; cy < ncy; ++cy)
        for (int col = 0; col < 2; ++col) {
            a.colour = col;
            a.update = !(cy == 0 && col == 0);
            a.first = cy == 0;
            a.keep = cy + 1 < ncy;
            a.send = a.keep || col == 0;
            a.rin = cy == 0 ? (const float4 *)r : nullptr;
            k_sap_step<<<nblk / 2, kSapSites, 0, s>>>(a);
            HIP_CHECK(hipGetLastError());
        }
    k_sap_unorder<<<grid_for(vh), kBlock, 0, s>>>(c->g, nb4, (float4 *)psi, pb);
    HIP_CHECK(hipGetLastError());
}

}  // namespace dl
