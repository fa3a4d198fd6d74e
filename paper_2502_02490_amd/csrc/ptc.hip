// Gauge-covariant parallel-transport convolution (PTC) network used as a learned
// preconditioner (a reading of the learned part; the paper has none):
//   y_c(x) = sum_{c'} sum_p W[p, c, c'] (T_p x_{c'})(x),   p in (0, +0, -0, +1, -1, +2, -2, +3, -3),
//   T_{+mu} psi(x) = V_mu(x) b+ psi(x + mu),  T_{-mu} psi(x) = V_mu(x - mu)^dag b- psi(x - mu),
// W a complex 4x4 spin matrix per (path, output, input) channel.  Activations are FP32 NATIVE
// full-lattice fields, one per channel; the working weights are BF16 (rounded from FP32 master
// weights); every product accumulates in FP32.
//   forward:   one thread per site, all output channels accumulated in registers;
//   backward:  input gradient = the same layer kernel with weights W'[q][c'][c] = W[adj q][c][c']^dag
//              (spin matrices commute with the transports, and T_p^dag = T_{adj p});
//              weight gradient dL/dW*[p,c,c'] = sum_{x, colour} g_c(x) (T_p x_{c'})(x)^dag, a
//              contraction over the sites on the matrix cores, reduced over tiles in index order
//              (deterministic);
//   Adam on (Re W, Im W) with FP32 state.
#include <cmath>
#include <vector>

#include "blas.h"
#include "dirac_ops.h"
#include "ptc.h"

namespace dl {
namespace {

constexpr int kPaths = 9;
constexpr int kTile = 64;  // sites per tile of the weight-gradient kernel

struct PtcGeom {
    Geom g;
    const float4 *flinks[2];  // per parity: full FP32 links F = e^{i omega} U, [8 dir][5 planes] blocked
};

// The network's transports use the links with the U(1) and boundary phase folded in and the
// third row rebuilt, F_n(x) = e^{i omega_n(x)} U_n(x) as 9 complex numbers (row-major, 18 floats
// in 5 planes of float4, the last two floats unused), built once per context: the hop kernel's
// compressed form would cost a sincos and a cross product in every one of the 9 * c_in
// transports of a site.
constexpr int kFullPlanes = 5;

__global__ void k_full_links(Geom g, int p, const float4 *__restrict__ links, const float *__restrict__ omega,
                             float4 *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.vh) return;
    const size_t vhp = (size_t)g.vhp;
#pragma unroll 1
    for (int n = 0; n < 8; ++n) {
        const float4 *lb = site_ptr(links + (size_t)n * 3 * vhp, (uint32_t)i, 3);
        float u12[12];
#pragma unroll
        for (int k = 0; k < 3; ++k) Lk<float>::unpack(lb[k * kSB], u12 + 4 * k);
        C<float> u[6], r2[3];
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = mk(u12[2 * k], u12[2 * k + 1]);
        third_row(u, r2);
        float si, co;
        sc(omega[(size_t)n * vhp + i], si, co);
        const C<float> ph = mk(co, si);
        float f[20];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const C<float> v = ph * u[k];
            f[2 * k] = v.r;
            f[2 * k + 1] = v.i;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const C<float> v = ph * r2[k];
            f[12 + 2 * k] = v.r;
            f[13 + 2 * k] = v.i;
        }
        f[18] = f[19] = 0.f;
        float4 *ob = site_ptr(out + (size_t)n * kFullPlanes * vhp, (uint32_t)i, kFullPlanes);
#pragma unroll
        for (int k = 0; k < kFullPlanes; ++k) ob[k * kSB] = make_float4(f[4 * k], f[4 * k + 1], f[4 * k + 2], f[4 * k + 3]);
    }
}

// Storage of an activation channel: a full NATIVE field (both parities), FP32 (six 16-byte
// planes of 4 reals per site) or BF16 (three planes of 8 reals).  The network's input and
// output and every gradient are FP32; its hidden activations are BF16, the precision in which
// the matrix cores read them anyway.
template <typename A> struct Act;
template <> struct Act<float> {
    using vec = float4;
    static constexpr int planes = 6;
};
template <> struct Act<__hip_bfloat16> {
    using vec = uint4;
    static constexpr int planes = 3;
};
using bf16s = __hip_bfloat16;
template <typename A> HD size_t chan_vecs(int vhp) { return (size_t)2 * Act<A>::planes * vhp; }  // per channel
template <typename A> HD size_t half_vecs(int vhp) { return (size_t)Act<A>::planes * vhp; }      // per parity

// Raw data of one transport: the (neighbour's) spinor and, for a hop, the full link.
template <typename A> struct TRaw {
    typename Act<A>::vec sp[Act<A>::planes];
    float4 lk[kFullPlanes];
};

// Load what T_path x_c needs at site (p, i) with coordinates x: the spinor, and the link of a hop (zero for the
// unshifted path).  Every field of r is written on every path, so the compiler keeps r in registers.
template <typename A>
DEV void spinor_load(const PtcGeom &a, const typename Act<A>::vec *xc, int p, uint32_t i, const int x[4], int path,
                     typename Act<A>::vec *sp) {
    constexpr int NP = Act<A>::planes;
    const size_t hv = half_vecs<A>(a.g.vhp);
    const int n = path - 1;  // direction index 2 mu + back (path > 0)
    const int mu = n >> 1, back = n & 1;
    int y[4] = {x[0], x[1], x[2], x[3]};
    if (path > 0) {
        const int xm = mu == 0 ? x[0] : mu == 1 ? x[1] : mu == 2 ? x[2] : x[3];
        const int Lm = mu == 0 ? a.g.L[0] : mu == 1 ? a.g.L[1] : mu == 2 ? a.g.L[2] : a.g.L[3];
        const int xn = back ? (xm == 0 ? Lm - 1 : xm - 1) : (xm + 1 == Lm ? 0 : xm + 1);
        const bool cross = back ? xm == 0 : xm + 1 == Lm;
        if (mu == 0) y[0] = xn; else if (mu == 1) y[1] = xn; else if (mu == 2) y[2] = xn; else y[3] = xn;
        y[1] = cstar_x1(a.g, mu, cross, y[1]);  // C*: into the mirror copy
    }
    const uint32_t j = path > 0 ? (uint32_t)half_index(a.g, y) : i;
    const int q = path > 0 ? 1 - p : p;
    const typename Act<A>::vec *b = site_ptr(xc + q * hv, j, NP);
#pragma unroll
    for (int k = 0; k < NP; ++k) sp[k] = b[k * kSB];
}
DEV void full_link_load(const PtcGeom &a, int p, uint32_t i, int path, float4 *lk) {
    if (path > 0) {
        const float4 *lb = site_ptr(a.flinks[p] + (size_t)(path - 1) * kFullPlanes * a.g.vhp, i, kFullPlanes);
#pragma unroll
        for (int k = 0; k < kFullPlanes; ++k) lk[k] = ld_stream(lb + k * kSB);  // read-once stream
    } else {
#pragma unroll
        for (int k = 0; k < kFullPlanes; ++k) lk[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}
template <typename A>
DEV void transport_load(const PtcGeom &a, const typename Act<A>::vec *xc, int p, uint32_t i, const int x[4], int path,
                        TRaw<A> &r) {
    spinor_load<A>(a, xc, p, i, x, path, r.sp);
    full_link_load(a, p, i, path, r.lk);
}

DEV void unpack4(const float4 *v, int nv, float *o) {
#pragma unroll
    for (int k = 0; k < nv; ++k) {
        o[4 * k] = v[k].x;
        o[4 * k + 1] = v[k].y;
        o[4 * k + 2] = v[k].z;
        o[4 * k + 3] = v[k].w;
    }
}
DEV void unpack_sp(const float4 *v, float *o) { unpack4(v, 6, o); }
DEV void unpack_sp(const uint4 *v, float *o) {
#pragma unroll
    for (int k = 0; k < 3; ++k) St<__hip_bfloat16>::unpack(v[k], o + 8 * k);
}

template <typename V>
DEV void transport_compute(const V *raw, const float4 *lk, int path, C<float> t[12]) {
    float sp[24];
    unpack_sp(raw, sp);
    if (path == 0) {
#pragma unroll
        for (int k = 0; k < 12; ++k) t[k] = mk(sp[2 * k], sp[2 * k + 1]);
        return;
    }
    float lf[20];
    unpack4(lk, kFullPlanes, lf);
    C<float> f[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) f[k] = mk(lf[2 * k], lf[2 * k + 1]);
    C<float> ps[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) ps[k] = mk(sp[2 * k], sp[2 * k + 1]);
    // one branch for the whole spinor (it is uniform where the path is)
    if (((path - 1) & 1) != 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                C<float> acc = mk(0.f, 0.f);
#pragma unroll
                for (int b = 0; b < 3; ++b) cmadd(acc, f[3 * b + a], ps[3 * s + b]);  // conj(F_ba) psi_b
                t[3 * s + a] = acc;
            }
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                C<float> acc = mk(0.f, 0.f);
#pragma unroll
                for (int b = 0; b < 3; ++b) madd(acc, f[3 * a + b], ps[3 * s + b]);
                t[3 * s + a] = acc;
            }
    }
}

// t = T_path x_c at site (p, i)
template <typename A>
DEV void transport_site(const PtcGeom &a, const typename Act<A>::vec *xc, int p, uint32_t i, const int x[4],
                        int path, C<float> t[12]) {
    TRaw<A> r;
    transport_load<A>(a, xc, p, i, x, path, r);
    transport_compute(r.sp, r.lk, path, t);
}

// Store 12 consecutive reals (reals 12 h .. 12 h + 11 of the 24, half h of the spinor) of site
// i of parity p of channel c.
DEV void store_half(float4 *base, int vhp, int c, int p, uint32_t i, int h, const float r[12]) {
    float4 *dst = site_ptr(base + c * chan_vecs<float>(vhp) + p * half_vecs<float>(vhp), i, 6) + 3 * h * kSB;
#pragma unroll
    for (int k = 0; k < 3; ++k) st_stream(dst + k * kSB, make_float4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]));
}
DEV void store_half(uint4 *base, int vhp, int c, int p, uint32_t i, int h, const float r[12]) {
    uint4 *site = site_ptr(base + c * chan_vecs<bf16s>(vhp) + p * half_vecs<bf16s>(vhp), i, 3);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int r0 = 12 * h + 4 * k;  // plane r0 / 8, half (r0 % 8) / 4 of it
        uint2 *dst = reinterpret_cast<uint2 *>(site + (r0 >> 3) * kSB) + ((r0 >> 2) & 1);
        const uint32_t lo = St<bf16s>::rne(r[4 * k]) | (St<bf16s>::rne(r[4 * k + 1]) << 16);
        const uint32_t hi = St<bf16s>::rne(r[4 * k + 2]) | (St<bf16s>::rne(r[4 * k + 3]) << 16);
        st_stream(dst, make_uint2(lo, hi));
    }
}

// ------------------------------------------------------------------ matrix-core layer
// The layer as a real GEMM on the 16x16x32 BF16 matrix cores (FP32 accumulation):
//   rows    m = 8 c + 2 sigma + ri_out          (output channel, spin, re/im)
//   columns n = (site, colour)                  (16 sites of a wavefront per tile, one colour per tile)
//   depth   k = 8 pair + 2 tau + ri_in,  pair = path * n_in + c' (path major: the four pairs of
//           a K step share one link, which the four lane groups load in one instruction; the
//           input-channel-major order was measured 1.5x slower, and channel groups outermost
//           with the paths into one neighbouring block consecutive fetched 5 % fewer bytes in
//           the same time)
// with the real embedding of the complex weights: (re, re) = (im, im) = Re W, (re, im) = -Im W,
// (im, re) = Im W.  A K step of 32 holds four (path, c') pairs; the lanes with k group g = lane / 16
// compute the transport T_path x_c' of pair 4 q + g at their site, and its 4 spins of colour a
// are exactly their 8 B-operand values for colour tile a, so each transport is computed once.
// The A operand (weights) is prepared once per weight update in the lane order of the
// instruction (row lane % 16, depth 8 (lane / 16) + j) and staged in LDS per work-group.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// A fragments of one layer: Af[(q * nm + t) * 64 + lane] = 8 BF16 values (uint4), q < nk, t < nm.
// W holds BF16 (re, im) pairs [9][nout][nin][4][4].
__global__ void k_ptc_afrag(int nin, int nout, int nk, int nm, const uint32_t *__restrict__ W,
                            uint4 *__restrict__ Af) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nk * nm * 64) return;
    const int lane = e & 63, t = (e >> 6) % nm, q = (e >> 6) / nm;
    const int m = 16 * t + (lane & 15), pair = 4 * q + (lane >> 4);
    const int c = m >> 3, sg = (m >> 1) & 3, rio = m & 1;
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (c < nout && pair < kPaths * nin) {
        const int path = pair / nin, cp = pair % nin;
        const uint32_t *w = W + ((size_t)(path * nout + c) * nin + cp) * 16 + sg * 4;
#pragma unroll
        for (int tau = 0; tau < 4; ++tau) {
            const uint32_t re = w[tau] & 0xffffu, im = w[tau] >> 16;
            // (ri_out, ri_in = 0) and (ri_out, ri_in = 1)
            const uint32_t lo = rio ? im : re, hi = rio ? re : (im ^ 0x8000u);
            v[tau] = lo | (hi << 16);
        }
    }
    Af[e] = make_uint4(v[0], v[1], v[2], v[3]);
}

// A fragments of the contraction z = W x of a contract-first last layer (one output channel) on
// the 16x16x16 BF16 matrix cores: rows m = 8 p + 2 sigma + ri_out (path, spin, re/im; 5 tiles,
// the last half empty), depth k = 8 c' + 2 tau + ri_in (the previous layer's output rows, NM tiles
// of 16).  Az[(tz * nm + t) * 64 + lane] = 4 BF16 values (uint2): row 16 tz + lane % 16, depth
// 16 t + 4 (lane / 16) + j.  W holds BF16 (re, im) pairs [9][1][nin][4][4].
constexpr int kZTiles = 5;
__global__ void k_ptc_zfrag(int nin, int nm, const uint32_t *__restrict__ W, uint2 *__restrict__ Az) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kZTiles * nm * 64) return;
    const int lane = e & 63, t = (e >> 6) % nm, tz = (e >> 6) / nm;
    const int m = 16 * tz + (lane & 15);
    const int path = m >> 3, sg = (m >> 1) & 3, rio = m & 1;
    uint32_t h[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = 16 * t + 4 * (lane >> 4) + j;
        const int cp = k >> 3, tau = (k >> 1) & 3, rii = k & 1;
        if (path < kPaths && cp < nin) {
            const uint32_t w = W[((size_t)path * nin + cp) * 16 + sg * 4 + tau];
            const uint32_t re = w & 0xffffu, im = w >> 16;
            // (re, re) = (im, im) = Re W, (re, im) = -Im W, (im, re) = Im W
            h[j] = rio == rii ? re : (rio ? im : (im ^ 0x8000u));
        }
    }
    Az[e] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
}

constexpr int kEoIn = 1, kEoOut = 2;  // even-odd deployment flags of the layer kernel

// One layer on the matrix cores.  Persistent: the grid's work-groups (4 wavefronts, 16 sites
// each) sweep the 64-site blocks of both parities; the A fragments are staged once per
// work-group.  NIN input channels, NM = ceil(8 NOUT / 16) row tiles.
// ZOUT: the next layer is a contract-first last layer; its contractions z_p = sum_c' W[p][c'] y_c'
// (p < 9) are formed from this layer's accumulators in registers -- the 16x16 accumulator tile t
// of a lane is, rounded to BF16, its B operand of depth step t on the 16x16x16 instruction -- and
// written to zout as 9 channels; y itself is written only when store_y is set.
// Work-groups a compute unit holds: the input gradient of a hidden first layer (8 -> 1 channels: 140 registers) fits
// three times (1.77 -> 1.56 ms at 32^3 x 64; four with a few spills 1.63); the others have more registers or little to wait for.
constexpr int layer_groups(int nin, int nm, bool zout) { return nin >= 4 && nm == 1 && !zout ? 3 : 2; }

template <int NIN, int NM, bool ZOUT, typename AI, typename AO>
__global__ __launch_bounds__(256, layer_groups(NIN, NM, ZOUT)) void k_ptc_layer_mfma(PtcGeom a, int nout, const uint4 *__restrict__ Af,
                                                        const typename Act<AI>::vec *__restrict__ xin,
                                                        typename Act<AO>::vec *__restrict__ yout,
                                                        const uint2 *__restrict__ Az, float4 *__restrict__ zout,
                                                        int store_y, int eo) {
    constexpr int NPAIR = kPaths * NIN, NK = (NPAIR + 3) / 4;
    __shared__ uint4 af[NK * NM * 64];
    for (int e = threadIdx.x; e < NK * NM * 64; e += 256) af[e] = Af[e];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, sl = lane & 15;
    const int nbp = (a.g.vh + 63) / 64;
    const size_t chin = chan_vecs<AI>(a.g.vhp);
#pragma nounroll
    for (int blk = blockIdx.x; blk < 2 * nbp; blk += gridDim.x) {
        const int p = blk >= nbp;
        const int b = blk - p * nbp;
        const int i = b * 64 + wave * 16 + sl;
        const bool on = i < a.g.vh;
        // A lane past the end of the lattice computes the transports of the last site: the
        // matrix-core output column of a site depends on that site's B column alone, and its
        // results are not stored.  Depth slots past the last (path, c') pair load pair NPAIR - 1;
        // their A fragments are zero, and the loaded values are finite.
        const uint32_t ic = on ? (uint32_t)i : (uint32_t)(a.g.vh - 1);
        int x[4];
        site_coords(a.g, (int)ic, p, x);
        f32x4_t acc[NM][3];
#pragma unroll
        for (int t = 0; t < NM; ++t)
#pragma unroll
            for (int col = 0; col < 3; ++col) acc[t][col] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        auto mul = [&](int q, const C<float> tr[12]) {
            bf16x8_t b[3];
#pragma unroll
            for (int col = 0; col < 3; ++col) {
#pragma unroll
                for (int tau = 0; tau < 4; ++tau) {
                    b[col][2 * tau] = (__bf16)tr[3 * tau + col].r;  // round to nearest even
                    b[col][2 * tau + 1] = (__bf16)tr[3 * tau + col].i;
                }
            }
#pragma unroll
            for (int t = 0; t < NM; ++t) {
                const bf16x8_t A = __builtin_bit_cast(bf16x8_t, af[(q * NM + t) * 64 + lane]);
#pragma unroll
                for (int col = 0; col < 3; ++col)
                    acc[t][col] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, b[col], acc[t][col], 0, 0, 0);
            }
        };
        if constexpr (NIN >= 4) {
            // Whole K steps per path: the steps unrolled, so that direction and neighbour are known at compile time,
            // a link read once for the steps of its path, spinors two steps ahead.  32^3 x 64, 8 -> 8 channels with
            // contractions 2.09 -> 1.57 ms (5,350 -> 3,900 VALU instructions a 16-site tile, 63 % of the SIMD cycles;
            // without the scheduling fence, which keeps the loads ahead, 1.72), FP32 2.03 -> 1.77 ms (11 GB
            // fetched past L2 at 6 TB/s; taking the tiles in the order of the weight gradient or in
            // cubes per XCD fetches up to 15 % less in the same time).
            constexpr int QP = NIN / 4, NLK = QP == 1 ? 3 : 2;  // steps of a path; links held: of the paths of q .. q + 2
            typename Act<AI>::vec sp[3][Act<AI>::planes];
            float4 lk[NLK][kFullPlanes];
            auto load = [&](int q) {
                const int path = q / QP;
                spinor_load<AI>(a, xin + (size_t)(4 * (q % QP) + g) * chin, p, ic, x, path, sp[q % 3]);
                if (q % QP == 0) full_link_load(a, p, ic, path, lk[path % NLK]);
            };
            load(0);
            load(1);
#pragma unroll
            for (int q = 0; q < NK; ++q) {
                if (q + 2 < NK) load(q + 2);
                __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the step's arithmetic
                C<float> tr[12];
                transport_compute(sp[q % 3], lk[q / QP % NLK], q / QP, tr);
                mul(q, tr);
            }
        } else {
            auto pair_of = [&](int q) {
                const int pr = 4 * q + g;
                if constexpr (NPAIR % 4 != 0) return pr < NPAIR ? pr : NPAIR - 1;
                return pr;
            };
            auto load = [&](int q, TRaw<AI> &r) {
                const int pair = pair_of(q);
                transport_load<AI>(a, xin + (size_t)(pair % NIN) * chin, p, ic, x, pair / NIN, r);
            };
            auto step = [&](int q, const TRaw<AI> &r) {
                C<float> tr[12];
                transport_compute(r.sp, r.lk, pair_of(q) / NIN, tr);
                mul(q, tr);
            };
            // software pipeline over three register sets in turn: the loads of K step q + 2 are
            // issued before the transport and the matrix-core work of step q
            // kEoIn (a network's first layer, one channel): the input's odd half is zero, so at an even site every
            // path but the unshifted one transports zeros; its K steps after that of path 0 add exact zeros and are skipped
            const int nk = ((eo & kEoIn) && p == 0) ? (NIN + 3) / 4 : NK;
            TRaw<AI> ra, rb, rc;
            load(0, ra);
            if (1 < nk) load(1, rb);
#pragma nounroll
            for (int q = 0; q < nk; q += 3) {
                if (q + 2 < nk) load(q + 2, rc);
                step(q, ra);
                if (q + 1 < nk) {
                    if (q + 3 < nk) load(q + 3, ra);
                    step(q + 1, rb);
                }
                if (q + 2 < nk) {
                    if (q + 4 < nk) load(q + 4, rb);
                    step(q + 2, rc);
                }
            }
        }
        // lane (g, site) holds rows m = 16 t + 4 g + r, r < 4: channel 2 t + g / 2, spins
        // 2 (g & 1) + r / 2, re/im r & 1 -- twelve consecutive reals (three planes) of one spinor
        auto store_tile = [&](const f32x4_t (&v)[3], auto *base, int c) {
            float r[12];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int col = 0; col < 3; ++col) r[6 * (rr >> 1) + 2 * col + (rr & 1)] = v[col][rr];
            store_half(base, a.g.vhp, c, p, (uint32_t)i, g & 1, r);
        };
        if (!ZOUT || store_y) {
            if (on) {
#pragma unroll
                for (int t = 0; t < NM; ++t)
                    if (2 * t + (g >> 1) < nout) store_tile(acc[t], yout, 2 * t + (g >> 1));
            }
        }
        if constexpr (ZOUT) {
            // every lane takes part in the matrix-core steps; only the stores are masked.  One
            // output tile at a time keeps the extra accumulators at 12 registers.
            // kEoOut: only the even half of the network's output is wanted, which reads z_0 at even
            // sites and z_1 .. z_8 at odd ones
            const bool eo_out = (eo & kEoOut) != 0;
            s16x4_t yb[NM][3];
#pragma unroll
            for (int t = 0; t < NM; ++t)
#pragma unroll
                for (int col = 0; col < 3; ++col) {
                    bf16x4_t b;
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) b[rr] = (__bf16)acc[t][col][rr];
                    yb[t][col] = __builtin_bit_cast(s16x4_t, b);
                }
            const int ntz = eo_out && p == 0 ? 1 : kZTiles;
#pragma nounroll
            for (int tz = 0; tz < ntz; ++tz) {
                f32x4_t zacc[3];
#pragma unroll
                for (int col = 0; col < 3; ++col) zacc[col] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int t = 0; t < NM; ++t) {
                    const s16x4_t A = __builtin_bit_cast(s16x4_t, Az[(tz * NM + t) * 64 + lane]);
#pragma unroll
                    for (int col = 0; col < 3; ++col)
                        zacc[col] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, yb[t][col], zacc[col], 0, 0, 0);
                }
                const int pz = 2 * tz + (g >> 1);
                const bool want = !eo_out || (p == 0 ? pz == 0 : pz > 0);
                if (on && pz < kPaths && want) store_tile(zacc, zout, pz);
            }
        }
    }
}

// y(x) = sum_p (T_p z_p)(x): the transports of a contract-first last layer (one output channel),
// one thread per site of either parity, the nine terms added in path order in FP32.
__global__ __launch_bounds__(256) void k_ptc_tsum(PtcGeom a, int nparity, const float4 *__restrict__ z,
                                                  float4 *__restrict__ y) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nparity * a.g.vh) return;
    const int p = s >= a.g.vh;
    const uint32_t i = (uint32_t)(s - p * a.g.vh);
    int x[4];
    site_coords(a.g, (int)i, p, x);
    const size_t chz = chan_vecs<float>(a.g.vhp);
    C<float> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = mk(0.f, 0.f);
#pragma nounroll
    for (int path = 0; path < kPaths; ++path) {
        C<float> t[12];
        transport_site<float>(a, z + (size_t)path * chz, p, i, x, path, t);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            acc[k].r += t[k].r;
            acc[k].i += t[k].i;
        }
    }
    float4 *dst = site_ptr(y + p * half_vecs<float>(a.g.vhp), i, 6);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        st_stream(dst + k * kSB, make_float4(acc[2 * k].r, acc[2 * k].i, acc[2 * k + 1].r, acc[2 * k + 1].i));
}

// Weight gradients on the BF16 matrix cores.  With Q_p = T_{adj p} (the adjoint of T_p),
//   dL/dW*[p,c,c'][s][t] = sum_{x, colour} g_c(x)_s conj((T_p x_c')(x)_t)
//                        = sum_{x, colour} (Q_p g_c)(x)_s conj(x_c'(x)_t),
// so the transports may be taken of either factor.  The kernel calls the transported factor "far"
// (NT channels) and the other, read at its own site, "near" (NL channels):
//   a hidden or last layer takes far = g, near = x: x is the BF16 activation, exact on the matrix
//   cores, and the last layer (one output channel) needs 9 transports per site instead of 72;
//   the first layer takes far = x (one channel, 9 transports), near = g, both FP32.
// The contraction is a real GEMM per 64-site tile: rows (pair = path NT + channel, spin, re/im) of
// the transports, columns (near channel, spin, re/im), depth k = 64 colour + site; the four
// (re/im, re/im) products of an output are combined in the final reduction.  FP32 operands are
// split exactly into three BF16 parts (truncation: 8 + 8 + 8 bits), the second scaled by 2^8 and the third by 2^16
// so that they keep the exponent of the value (unscaled, the parts of values below 1e-33 are subnormal in BF16 and
// lose bits).  So every product is exact and only the FP32 accumulation rounds, as in an FP32 contraction; of the
// nine products of two split operands the last (2^-32 of the value) is left out.
//
// A work-group of eight wavefronts, one per compute unit, sweeps its tiles.  Per tile it transposes
// the near factor through LDS into registers (B operands, kept for all paths); per group of 8 pairs
// (64 rows) each wavefront forms one pair's transports at the 64 sites, splits them, exchanges
// re and im between neighbouring lanes so that a lane packs two sites, and writes them to LDS
// ([part][row][k]); then the wavefronts multiply.  LDS holds two such buffers used in turn, so a
// group costs one barrier, and the raw data of the next group is loaded before the current one is
// multiplied.  All nine paths of a tile run in one work-group (accumulators: 72 registers for 8 -> 8
// channels), so the near factor is read once and the far factor's neighbours meet in L2.
// The products of a group go to accumulators of their own, one for each power of 2^-8, and are added
// to the running ones in FP32, the smallest parts first: the matrix cores do not round their sums to nearest (a chain over all
// tiles drifted to 2.4e-6 of the result at 32^3 x 64).  The running sums are added to the work-group's
// slice every kFlush tiles; one lane owns each entry of a slice (no atomics, deterministic).
// Measured at 32^3 x 64 (FP32 vector contraction with the transports of x before -> now): 8 -> 8
// channels 9.5 -> 3.65 ms, 8 -> 1 3.3 -> 0.76 ms, 1 -> 8 1.65 -> 1.10 ms; errors against 64 bits
// 1.2-2.9e-7 -> 1.0-1.4e-7.  The 8 -> 8 kernel is bound by none of its parts alone: vector ALU 55 %
// busy (about 400 instructions per transport), matrix cores 18 %, 10 GB fetched; without cache
// misses it takes 10 % less, without the matrix instructions 15 %, without the link products 5 %.
template <int NT, int NL, bool NEARBF>
struct WgradShape {
    static constexpr int NPAIR = kPaths * NT;
    static constexpr int NG = (NPAIR + 7) / 8;                    // groups of 8 pairs
    static constexpr int NCT = NL == 8 ? 4 : NL == 4 ? 2 : 1;     // 16-column tiles
    static constexpr int LS = NEARBF ? 1 : 3;                     // parts of the near factor
    // wavefronts along the four row tiles of a group and along the column tiles (a split near factor
    // of 8 channels takes one column tile per wavefront, which fits the registers); with one column
    // tile half the wavefronts have nothing to multiply
    static constexpr int WR = !NEARBF && NCT == 4 ? 2 : 4, WC = NCT == 1 ? 1 : 8 / WR;
    static constexpr int RT = 4 / WR, CT = NCT / WC;
    static constexpr int SLICE = NG * RT * CT * 64 * WR * WC;     // float4 per work-group
};
constexpr int kWRow = 384;      // bytes of a row of 192 BF16 in LDS
constexpr int kWBuf = 3 * 64 * kWRow;
// Byte offset of depth k = 64 colour + 8 chunk + ... of a row: the eight 16-byte chunks of a colour are
// permuted by the row, so that the 16-byte reads of 16 rows (and the 4-byte writes of two adjacent
// rows) fall in distinct banks.
DEV int wgrad_at(int row, int col, int chunk) { return row * kWRow + 128 * col + 16 * (chunk ^ ((row >> 1) & 7)); }
constexpr int kFlush = 16;      // tiles between additions of the accumulators to the slice

// Order of the 64-site tiles of one parity: XCD k (work-groups k mod 8, which dispatch places there)
// walks the time slices of its eighth of the x1 range where that is whole blocks, so the
// neighbours of a tile are read by the same XCD within a few slices; otherwise it takes the k-th
// contiguous eighth of the blocks.  Steps whose block is nbp or more are skipped.
DEV int tile_order(const Geom &g, int per, int xcd, int j) {
    if (g.L[1] % 8 != 0 || (g.vh / (g.L[0] * 8)) % kTile != 0) return xcd * per + j;
    const int bps = g.vh / (g.L[0] * 8 * kTile);
    return ((j / bps) * 8 + xcd) * bps + j % bps;
}

// v = hi + 2^-8 mid + 2^-16 lo exactly, each with at most 8 significant bits (BF16 in the upper half word)
DEV void split3(float v, uint32_t o[3]) {
    o[0] = __float_as_uint(v) & 0xffff0000u;
    const float r1 = (v - __uint_as_float(o[0])) * 256.f;
    o[1] = __float_as_uint(r1) & 0xffff0000u;
    o[2] = __float_as_uint((r1 - __uint_as_float(o[1])) * 256.f);
}
DEV uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }  // upper halves
// the value of the neighbouring lane (lane ^ 1)
DEV float lane_swap(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, false));
}

template <int NT, int NL, bool NEARBF>
__global__ __launch_bounds__(512, 2) void k_ptc_wgrad(PtcGeom a, const float4 *__restrict__ far_,
                                                      const void *__restrict__ near_, float4 *__restrict__ part) {
    using W = WgradShape<NT, NL, NEARBF>;
    __shared__ __align__(16) unsigned char sm[2 * kWBuf];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool mul = wave < W::WR * W::WC;
    const int wr = (wave / W::WC) % W::WR, wc = wave % W::WC;
    const int xcd = (int)blockIdx.x & 7, nwg = (int)gridDim.x >> 3;
    const int nbp = a.g.vhp / kTile, per = (nbp + 7) >> 3;
    const size_t chf = chan_vecs<float>(a.g.vhp);
    float4 *slice = part + (size_t)blockIdx.x * W::SLICE + tid;
    f32x4_t acc[W::NG][W::RT][W::CT];
    bool first = true, negate = (blockIdx.x & 8) != 0;
    int since = 0, buf = 0;
    auto clear = [&]() {
#pragma unroll
        for (int g = 0; g < W::NG; ++g)
#pragma unroll
            for (int r = 0; r < W::RT; ++r)
#pragma unroll
                for (int c = 0; c < W::CT; ++c) acc[g][r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto flush = [&]() {
        if (mul) {
#pragma unroll
            for (int g = 0; g < W::NG; ++g)
#pragma unroll
                for (int r = 0; r < W::RT; ++r)
#pragma unroll
                    for (int c = 0; c < W::CT; ++c) {
                        float4 *d = slice + ((g * W::RT + r) * W::CT + c) * (64 * W::WR * W::WC);
                        const f32x4_t v = acc[g][r][c];
                        const float4 o = first ? make_float4(0.f, 0.f, 0.f, 0.f) : *d;
                        *d = make_float4(o.x + v[0], o.y + v[1], o.z + v[2], o.w + v[3]);
                    }
        }
        clear();
        first = false;
        since = 0;
    };
    clear();
    // The lane's site of the tile being loaded (a lane past the end takes the last site: the near
    // factor is zero there) and the raw data of its next transport.
    int i = 0, x[4], lp = 0, lbase = 0;
    TRaw<float> raw;
    // With few groups per tile the near factor's loads would stall every tile: its raw data is loaded one tile
    // ahead as well (two neighbouring sites per thread of the first 32 NL threads).
    constexpr bool AHEAD = W::NG <= 2;
    using NV = typename Act<std::conditional_t<NEARBF, bf16s, float>>::vec;
    constexpr int NNP = NEARBF ? 3 : 6;
    const int nc = tid >> 5, sp = tid & 31;
    NV n0[AHEAD ? NNP : 1], n1[AHEAD ? NNP : 1];
    auto near_at = [&](int p, int base) {
        using A = std::conditional_t<NEARBF, bf16s, float>;
        return site_ptr((const NV *)near_ + nc * chan_vecs<A>(a.g.vhp) + p * half_vecs<A>(a.g.vhp),
                        (uint32_t)(base + 2 * sp), NNP);
    };
    auto load_near = [&]() {
        if (nc < NL) {
            const NV *q = near_at(lp, lbase);
#pragma unroll
            for (int k = 0; k < NNP; ++k) {
                n0[k] = q[k * kSB];
                n1[k] = q[k * kSB + 1];
            }
        }
    };
    auto next_tile = [&](int j) {  // the first step at or after j with a block of the lattice
        for (; j < 2 * per; j += nwg) {
            lp = j >= per;
            const int blk = tile_order(a.g, per, xcd, j - lp * per);
            if (blk >= nbp) continue;
            lbase = blk * kTile;
            i = min(lbase + lane, a.g.vh - 1);
            site_coords(a.g, i, lp, x);
            break;
        }
        return j;
    };
    // LDS offsets that do not change: this lane's words of the four spins' rows of its pair, and its A
    // operand rows (depth chunks 0..3 of a colour; chunks 4..7 sit 64 bytes away, across the swizzle)
    int wofs[4], aofs[W::RT];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
        wofs[sp] = wgrad_at(8 * wave + 2 * sp + (lane & 1), 0, lane >> 3) + 4 * ((lane >> 1) & 3);
#pragma unroll
    for (int r = 0; r < W::RT; ++r) aofs[r] = wgrad_at(16 * (wr * W::RT + r) + (lane & 15), 0, lane >> 4);
    auto load = [&](int grp) {
        const int pair = 8 * grp + wave;
        if (pair < W::NPAIR)
            transport_load<float>(a, far_ + (pair % NT) * chf, lp, (uint32_t)i, x, pair / NT, raw);
    };
    int j = next_tile((int)blockIdx.x >> 3);
    if (j < 2 * per) load(0);
    if constexpr (AHEAD) {
        if (j < 2 * per) load_near();
    }
#pragma nounroll
    while (j < 2 * per) {
        const int p = lp, base = lbase;
        int jn = j;
        // Every other tile takes the near factor negated and its products subtracted: the matrix cores
        // round their sums downwards, and the bias of the two kinds cancels.
        const float sign = negate ? -1.f : 1.f;
        const uint32_t flip = negate ? 0x80008000u : 0u;
        negate = !negate;
        // the near factor, two neighbouring sites per thread: [part][column][k]; sites past the end are zero
        const int s0 = base + 2 * sp;
        if (nc < NL) {
            const bool on0 = s0 < a.g.vh, on1 = s0 + 1 < a.g.vh;
            const NV *q = near_at(p, base);
            unsigned char *dst = sm + buf * kWBuf + 4 * (sp & 3);
            // real r = 6 t + 2 colour + ri of the spinor is column 2 t + ri, depth 64 colour + site
            auto put = [&](int part_, int r, uint32_t w) {
                *reinterpret_cast<uint32_t *>(
                    dst + part_ * 64 * kWRow + wgrad_at(8 * nc + 2 * (r / 6) + (r & 1), (r % 6) >> 1, sp >> 2)) = w ^ flip;
            };
            if constexpr (NEARBF) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint4 u0 = AHEAD ? n0[AHEAD ? k : 0] : q[k * kSB], u1 = AHEAD ? n1[AHEAD ? k : 0] : q[k * kSB + 1];
                    const uint32_t w0[4] = {u0.x, u0.y, u0.z, u0.w}, w1[4] = {u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const uint32_t v0 = on0 ? w0[m] : 0u, v1 = on1 ? w1[m] : 0u;
                        put(0, 8 * k + 2 * m, __builtin_amdgcn_perm(v1, v0, 0x05040100u));  // lower halves
                        put(0, 8 * k + 2 * m + 1, pack_hi(v0, v1));
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const float4 u0 = AHEAD ? n0[AHEAD ? k : 0] : q[k * kSB], u1 = AHEAD ? n1[AHEAD ? k : 0] : q[k * kSB + 1];
                    const float f0[4] = {u0.x, u0.y, u0.z, u0.w}, f1[4] = {u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        uint32_t y0[3], y1[3];
                        split3(on0 ? f0[m] : 0.f, y0);
                        split3(on1 ? f1[m] : 0.f, y1);
#pragma unroll
                        for (int q3 = 0; q3 < 3; ++q3) put(q3, 4 * k + m, pack_hi(y0[q3], y1[q3]));
                    }
                }
            }
        }
        __syncthreads();
        bf16x8_t nb[W::LS][W::CT][6];
#pragma unroll
        for (int l = 0; l < W::LS; ++l)
#pragma unroll
            for (int c = 0; c < W::CT; ++c)
#pragma unroll
                for (int ks = 0; ks < 6; ++ks)
                    nb[l][c][ks] = *reinterpret_cast<const bf16x8_t *>(
                        sm + buf * kWBuf + 64 * l * kWRow +
                        wgrad_at(16 * (wc * W::CT + c) + (lane & 15), ks >> 1, 4 * (ks & 1) + (lane >> 4)));
        buf ^= 1;
#pragma unroll
        for (int grp = 0; grp < W::NG; ++grp) {
            if (8 * grp + wave < W::NPAIR) {
                C<float> t[12];
                transport_compute(raw.sp, raw.lk, (8 * grp + wave) / NT, t);
                // an even lane packs the real parts of its own and the next site (row 2 s), an odd lane
                // the imaginary parts of the previous and its own site (row 2 s + 1)
                const bool odd = (lane & 1) != 0;
                const uint32_t sel = odd ? 0x03020706u : 0x07060302u;
                unsigned char *dst = sm + buf * kWBuf;
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    const float own = odd ? t[k].i : t[k].r, oth = lane_swap(odd ? t[k].r : t[k].i);
                    uint32_t y0[3], y1[3];
                    split3(own, y0);
                    split3(oth, y1);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        *reinterpret_cast<uint32_t *>(dst + wofs[k / 3] + 64 * q * kWRow + 128 * (k % 3)) =
                            __builtin_amdgcn_perm(y1[q], y0[q], sel);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (grp + 1 < W::NG) {
                load(grp + 1);
            } else {
                jn = next_tile(j + nwg);
                if (jn < 2 * per) {
                    load(0);
                    if constexpr (AHEAD) load_near();
                }
            }
            __syncthreads();
            // row tiles holding no pair of the last group are skipped (their rows were not written)
            constexpr int kLast = W::NPAIR - 8 * (W::NG - 1);
            const int rtiles = grp + 1 < W::NG ? 4 : (kLast + 1) / 2;
#pragma unroll
            for (int r = 0; r < W::RT; ++r) {
                if (!mul || wr * W::RT + r >= rtiles) continue;
                // v[n]: the products of weight 2^-8n
                constexpr int NV = W::LS > 1 ? 4 : 3;
                f32x4_t v[NV][W::CT];
#pragma unroll
                for (auto &u : v)
#pragma unroll
                    for (auto &w : u) w = f32x4_t{0.f, 0.f, 0.f, 0.f};
                const unsigned char *a0 = sm + buf * kWBuf + aofs[r], *a1 = sm + buf * kWBuf + (aofs[r] ^ 64);
#pragma unroll
                for (int q = 2; q >= 0; --q) {
#pragma unroll
                    for (int ks = 0; ks < 6; ++ks) {
                        const bf16x8_t A = *reinterpret_cast<const bf16x8_t *>(
                            (ks & 1 ? a1 : a0) + 64 * q * kWRow + 128 * (ks >> 1));
#pragma unroll
                        for (int l = W::LS - 1; l >= 0; --l) {
                            if (q + l == 4) continue;
#pragma unroll
                            for (int c = 0; c < W::CT; ++c)
                                v[q + l][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, nb[l][c][ks], v[q + l][c], 0, 0, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // bounds the LDS reads in flight (registers)
                }
#pragma unroll
                for (int c = 0; c < W::CT; ++c) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float u = v[NV - 1][c][e];
#pragma unroll
                        for (int n = NV - 2; n >= 0; --n) u = fmaf(u, 0x1p-8f, v[n][c][e]);
                        acc[grp][r][c][e] = fmaf(sign, u, acc[grp][r][c][e]);
                    }
                }
            }
            buf ^= 1;
        }
        if (++since == kFlush) flush();
        j = jn;
    }
    if (since || first) flush();
}

// out[k] += the weight gradients from the slices of k_ptc_wgrad.  A work-group of 256 threads takes
// 16 consecutive float4 of the slices (one lane group of a 16 x 16 accumulator tile: 4
// rows x 16 columns); 16 strands of threads sum the slices in FP64 and are added in order
// (deterministic), then the four (re/im, re/im) sums of each of the 16 outputs are combined.
template <int NT, int NL, bool NEARBF>
__global__ __launch_bounds__(256) void k_ptc_reduce(int nwg, const float4 *__restrict__ part, float2 *__restrict__ out) {
    using W = WgradShape<NT, NL, NEARBF>;
    constexpr int SL = 16;
    __shared__ double sum[SL][4][16];
    constexpr int TL = 64 * W::WR * W::WC;  // float4 of one accumulator tile of every wavefront
    const int f0 = (int)blockIdx.x * 16;
    const int j = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int tl = f0 / TL, wave = (f0 % TL) >> 6, lg = (f0 >> 4) & 3;
    const int ct = (wave % W::WC) * W::CT + tl % W::CT;
    const int rt = (wave / W::WC) * W::RT + (tl / W::CT) % W::RT, gl = tl / (W::CT * W::RT);
    const int pair = 8 * gl + 2 * rt + (lg >> 1);
    if (pair >= W::NPAIR) return;  // uniform over the work-group
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int b = sl; b < nwg; b += SL) {
        const float4 q = part[(size_t)b * W::SLICE + f0 + j];
        v[0] += q.x;
        v[1] += q.y;
        v[2] += q.z;
        v[3] += q.w;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[sl][r][j] = v[r];
    __syncthreads();
    if (threadIdx.x < 64) {
        const int r = threadIdx.x >> 4;
        double s = sum[0][r][j];
        for (int b = 1; b < SL; ++b) s += sum[b][r][j];
        sum[0][r][j] = s;
    }
    __syncthreads();
    if (threadIdx.x >= 16) return;
    // rows 2 rr + ri (far spin 2 (lg & 1) + rr), columns 2 cp + ri (near channel and spin)
    const int rr = threadIdx.x >> 3, cp = threadIdx.x & 7;
    const int cl = 2 * ct + (cp >> 2), sn = cp & 3, sf = 2 * (lg & 1) + rr;
    if (cl >= NL) return;
    const double re = sum[0][2 * rr][2 * cp] + sum[0][2 * rr + 1][2 * cp + 1];
    const double im = sum[0][2 * rr + 1][2 * cp] - sum[0][2 * rr][2 * cp + 1];  // Im(far conj(near))
    const int path = pair / NT, ch = pair % NT;
    size_t k;
    double sg = 1.0;
    if (NEARBF) {  // far = g (NT = c_out), transported along the adjoint path; near = x (NL = c_in)
        const int pa = path == 0 ? 0 : ((path - 1) ^ 1) + 1;
        k = ((size_t)(pa * NT + ch) * NL + cl) * 16 + sf * 4 + sn;
    } else {  // far = x (one channel), near = g (NL = c_out): g conj(x)
        k = ((size_t)path * NL + cl) * 16 + sn * 4 + sf;
        sg = -1.0;
    }
    out[k].x += (float)re;
    out[k].y += (float)(sg * im);
}

// Adam on n real parameters (interleaved re, im); writes the BF16 working copy
// omb1 = 1 - b1 and omb2 = 1 - b2 come rounded once from their exact values: 1 - b2 formed in FP32
// from the rounded b2 = 0.999f would be 1.3e-5 off in relative terms.
__global__ void k_adam(int n, float *__restrict__ w, const float *__restrict__ grad_conj, float *__restrict__ m,
                       float *__restrict__ v, uint16_t *__restrict__ wbf, float lr, float b1, float omb1, float b2,
                       float omb2, float eps, float c1, float c2) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float g = 2.0f * grad_conj[k];  // dL/d(Re W) = 2 Re dL/dW*, dL/d(Im W) = 2 Im dL/dW*
    const float mk_ = b1 * m[k] + omb1 * g;
    const float vk = b2 * v[k] + omb2 * g * g;
    m[k] = mk_;
    v[k] = vk;
    const float nw = w[k] - lr * (mk_ / c1) / (sqrtf(vk / c2) + eps);
    w[k] = nw;
    wbf[k] = (uint16_t)St<__hip_bfloat16>::rne(nw);
}

__global__ void k_to_bf16(int n, const float *__restrict__ w, uint16_t *__restrict__ wbf) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) wbf[k] = (uint16_t)St<__hip_bfloat16>::rne(w[k]);
}

// W'[q][c'][c] = W[adj q][c][c']^dag (spin 4x4), on BF16 pairs (exact: a permutation and sign flips)
__global__ void k_adjoint_weights(int nout, int nin, const uint32_t *__restrict__ W, uint32_t *__restrict__ Wt) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int total = kPaths * nin * nout * 16;
    if (k >= total) return;
    const int st = k & 15, ss = st >> 2, tt = st & 3;
    int r = k >> 4;
    const int c = r % nout;  // Wt index [q][c'][c]: c fastest
    r /= nout;
    const int cp = r % nin;
    const int q = r / nin;
    const int adj[kPaths] = {0, 2, 1, 4, 3, 6, 5, 8, 7};
    const uint32_t w = W[((size_t)(adj[q] * nout + c) * nin + cp) * 16 + tt * 4 + ss];  // transpose
    Wt[k] = w ^ 0x80000000u;                                                              // conjugate
}

int compute_units() {
    static int n = 0;
    if (!n) {
        int dev = 0, v = 0;
        HIP_CHECK(hipGetDevice(&dev));
        HIP_CHECK(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        n = v > 0 ? v : 256;
    }
    return n;
}
int row_tiles(int nout) { return (8 * nout + 15) / 16; }
int k_steps(int nin) { return (kPaths * nin + 3) / 4; }
size_t afrag_count(int nin, int nout) { return (size_t)k_steps(nin) * row_tiles(nout) * 64; }
size_t zfrag_count(int nin) { return (size_t)kZTiles * row_tiles(nin) * 64; }

void build_zfrags(int nin, const uint32_t *W, uint2 *Az, hipStream_t s) {
    const int n = (int)zfrag_count(nin);
    k_ptc_zfrag<<<(n + 255) / 256, 256, 0, s>>>(nin, row_tiles(nin), W, Az);
    HIP_CHECK(hipGetLastError());
}

void build_afrags(int nin, int nout, const uint32_t *W, uint4 *Af, hipStream_t s) {
    const int n = (int)afrag_count(nin, nout);
    k_ptc_afrag<<<(n + 255) / 256, 256, 0, s>>>(nin, nout, k_steps(nin), row_tiles(nout), W, Af);
    HIP_CHECK(hipGetLastError());
}

// Storage of a layer's input and output: FP32 -> FP32 (the input-gradient pass, and a network of
// one layer), FP32 -> BF16 (the first layer), BF16 -> BF16 (the hidden layers).
enum class Io { F32, In, Mid };
// The optional ZOUT arguments (Az, z, store_y) select the variant that also forms the
// contractions of a contract-first last layer.
struct ZArgs {
    const uint2 *Az = nullptr;
    void *z = nullptr;
    bool store_y = true;
    int eo = 0;  // kEoIn, kEoOut
};
template <int NIN, int NM, bool ZOUT, typename AI, typename AO>
void launch_io(int grid, const PtcGeom &a, int nout, const uint4 *Af, const void *x, void *y, const ZArgs &zo,
               hipStream_t s) {
    k_ptc_layer_mfma<NIN, NM, ZOUT, AI, AO><<<grid, 256, 0, s>>>(
        a, nout, Af, (const typename Act<AI>::vec *)x, (typename Act<AO>::vec *)y, zo.Az, (float4 *)zo.z,
        zo.store_y ? 1 : 0, zo.eo);
}
template <int NIN, int NM>
void launch_layer(const PtcGeom &a, int nout, const uint4 *Af, const void *x, void *y, const ZArgs &zo, Io io,
                  hipStream_t s) {
    const int nblk = 2 * (int)((a.g.vh + 63) / 64);
    const int grid = std::min(nblk, layer_groups(NIN, NM, zo.z != nullptr) * compute_units());
    if (zo.z) {
        if (io == Io::In) launch_io<NIN, NM, true, float, bf16s>(grid, a, nout, Af, x, y, zo, s);
        else if (io == Io::Mid) launch_io<NIN, NM, true, bf16s, bf16s>(grid, a, nout, Af, x, y, zo, s);
        else throw Error(DIRAC_EUNSUPPORTED, "contract-first epilogue needs a BF16 layer output");
    } else {
        if (io == Io::In) launch_io<NIN, NM, false, float, bf16s>(grid, a, nout, Af, x, y, zo, s);
        else if (io == Io::Mid) launch_io<NIN, NM, false, bf16s, bf16s>(grid, a, nout, Af, x, y, zo, s);
        else launch_io<NIN, NM, false, float, float>(grid, a, nout, Af, x, y, zo, s);
    }
}
template <int NIN>
void launch_layer_nm(const PtcGeom &a, int nout, const uint4 *Af, const void *x, void *y, const ZArgs &zo, Io io,
                     hipStream_t s) {
    switch (row_tiles(nout)) {
        case 1: launch_layer<NIN, 1>(a, nout, Af, x, y, zo, io, s); break;
        case 2: launch_layer<NIN, 2>(a, nout, Af, x, y, zo, io, s); break;
        default: launch_layer<NIN, 4>(a, nout, Af, x, y, zo, io, s); break;
    }
}
// y = layer(x) with the A fragments Af of a (nin -> nout) layer
void layer_dispatch(const PtcGeom &a, int nin, int nout, const void *x, const uint4 *Af, void *y, Io io, hipStream_t s,
                    const ZArgs &zo = ZArgs()) {
    switch (nin) {
        case 1: launch_layer_nm<1>(a, nout, Af, x, y, zo, io, s); break;
        case 2: launch_layer_nm<2>(a, nout, Af, x, y, zo, io, s); break;
        case 4: launch_layer_nm<4>(a, nout, Af, x, y, zo, io, s); break;
        case 8: launch_layer_nm<8>(a, nout, Af, x, y, zo, io, s); break;
        default: throw Error(DIRAC_EUNSUPPORTED, "PTC channel counts must be 1, 2, 4 or 8");
    }
    HIP_CHECK(hipGetLastError());
}
// Work-groups of the weight-gradient kernel, a multiple of 8 (the XCDs): one per compute unit (what its
// LDS allows), at most one per tile of an XCD.
int wgrad_groups(size_t vhp) {
    const size_t per = 2 * ((vhp / kTile + 7) / 8);
    return 8 * (int)std::max<size_t>(1, std::min(per, (size_t)compute_units() / 8));
}
template <int NT, int NL, bool NEARBF>
void launch_wgrad(const PtcGeom &a, const void *far_, const void *near_, void *part, float2 *out, hipStream_t s) {
    using W = WgradShape<NT, NL, NEARBF>;
    const int nwg = wgrad_groups(a.g.vhp);
    k_ptc_wgrad<NT, NL, NEARBF><<<nwg, 512, 0, s>>>(a, (const float4 *)far_, near_, (float4 *)part);
    k_ptc_reduce<NT, NL, NEARBF><<<W::SLICE / 16, 256, 0, s>>>(nwg, (const float4 *)part, out);
}
// Calls f with the shape of a layer's weight gradient: far and near channel counts, and whether the
// near factor is the BF16 activation of a hidden layer (else the first layer: far = x, near = g).
template <typename F> void wgrad_shape(int nin, int nout, bool x_bf16, F &&f) {
    auto near_of = [&](auto nt, int nl, auto bf) {
        switch (nl) {
            case 1: f(nt, std::integral_constant<int, 1>(), bf); break;
            case 2: f(nt, std::integral_constant<int, 2>(), bf); break;
            case 4: f(nt, std::integral_constant<int, 4>(), bf); break;
            case 8: f(nt, std::integral_constant<int, 8>(), bf); break;
            default: throw Error(DIRAC_EUNSUPPORTED, "PTC channel counts must be 1, 2, 4 or 8");
        }
    };
    if (!x_bf16) {
        require(nin == 1, "the first layer of a PTC network has one input channel", DIRAC_EUNSUPPORTED);
        near_of(std::integral_constant<int, 1>(), nout, std::false_type());
        return;
    }
    switch (nout) {
        case 1: near_of(std::integral_constant<int, 1>(), nin, std::true_type()); break;
        case 2: near_of(std::integral_constant<int, 2>(), nin, std::true_type()); break;
        case 4: near_of(std::integral_constant<int, 4>(), nin, std::true_type()); break;
        case 8: near_of(std::integral_constant<int, 8>(), nin, std::true_type()); break;
        default: throw Error(DIRAC_EUNSUPPORTED, "PTC output channels must be 1, 2, 4 or 8");
    }
}
// dW += the weight gradients of a layer with input x and output gradient g
void wgrad_dispatch(const PtcGeom &a, int nin, int nout, const void *x, bool x_bf16, const void *g, void *part,
                    float2 *dW, hipStream_t s) {
    wgrad_shape(nin, nout, x_bf16, [&](auto nt, auto nl, auto bf) {
        constexpr bool B = decltype(bf)::value;
        launch_wgrad<decltype(nt)::value, decltype(nl)::value, B>(a, B ? g : x, B ? x : g, part, dW, s);
    });
    HIP_CHECK(hipGetLastError());
}
size_t wgrad_part_bytes(size_t vhp, int nin, int nout, bool x_bf16) {
    size_t n = 0;
    wgrad_shape(nin, nout, x_bf16, [&](auto nt, auto nl, auto bf) {
        using W = WgradShape<decltype(nt)::value, decltype(nl)::value, decltype(bf)::value>;
        n = (size_t)wgrad_groups(vhp) * W::SLICE * sizeof(float4);
    });
    return n;
}

PtcGeom geom_of(dirac_ctx *c, hipStream_t s) {
    ensure_prec(c, DIRAC_F32, s);
    if (!c->ptc_links_ready) {
        const size_t per = (size_t)8 * kFullPlanes * c->g.vhp * sizeof(float4);
        for (int p = 0; p < 2; ++p) {
            c->ptc_links[p].alloc(per);
            k_full_links<<<grid_for(c->vh), kBlock, 0, s>>>(c->g, p, (const float4 *)c->f[DIRAC_F32].links[p].p,
                                                            (const float *)c->f[DIRAC_F32].omega[p].p,
                                                            (float4 *)c->ptc_links[p].p);
            HIP_CHECK(hipGetLastError());
        }
        c->ptc_links_ready = true;
    }
    PtcGeom a;
    a.g = c->g;
    for (int p = 0; p < 2; ++p) a.flinks[p] = (const float4 *)c->ptc_links[p].p;
    return a;
}

}  // namespace

size_t ptc_nweights(const dirac_ptc *n, int l) { return (size_t)kPaths * n->ch[l] * n->ch[l + 1] * 16; }

void ptc_alloc(dirac_ptc *n) {
    size_t tot = 0;
    for (int l = 0; l < n->nlayers; ++l) {
        n->off[l] = tot;
        tot += ptc_nweights(n, l);
    }
    n->total = tot;  // complex entries
    size_t fw = 0, fb = 0;
    for (int l = 0; l < n->nlayers; ++l) {
        n->afw_off[l] = fw;
        n->afb_off[l] = fb;
        fw += afrag_count(n->ch[l], n->ch[l + 1]);
        fb += afrag_count(n->ch[l + 1], n->ch[l]);
    }
    n->afw.alloc(fw * sizeof(uint4));
    n->afb.alloc(fb * sizeof(uint4));
    if (n->contract_last()) n->afz.alloc(zfrag_count(n->ch[n->nlayers - 1]) * sizeof(uint2));
    n->w.alloc(tot * 8);
    n->wbf.alloc(tot * 4);
    n->wt.alloc(tot * 4);
    n->grad.alloc(tot * 8);
    n->m.alloc(tot * 8);
    n->v.alloc(tot * 8);
    HIP_CHECK(hipMemset(n->w.p, 0, tot * 8));
    HIP_CHECK(hipMemset(n->wbf.p, 0, tot * 4));
    HIP_CHECK(hipMemset(n->grad.p, 0, tot * 8));
    HIP_CHECK(hipMemset(n->m.p, 0, tot * 8));
    HIP_CHECK(hipMemset(n->v.p, 0, tot * 8));
    n->step = 0;
}

// forward A fragments of every layer from the BF16 working weights
static void refresh_afrags(dirac_ptc *n, hipStream_t s) {
    for (int l = 0; l < n->nlayers; ++l)
        build_afrags(n->ch[l], n->ch[l + 1], (const uint32_t *)n->wbf.p + n->off[l], (uint4 *)n->afw.p + n->afw_off[l],
                     s);
    if (n->contract_last()) {
        const int l = n->nlayers - 1;
        build_zfrags(n->ch[l], (const uint32_t *)n->wbf.p + n->off[l], (uint2 *)n->afz.p, s);
    }
}

void ptc_refresh_bf16(dirac_ptc *n, hipStream_t s) {
    const int nr = (int)(2 * n->total);
    k_to_bf16<<<(nr + 255) / 256, 256, 0, s>>>(nr, (const float *)n->w.p, (uint16_t *)n->wbf.p);
    HIP_CHECK(hipGetLastError());
    refresh_afrags(n, s);
}

// Activation l is stored in BF16 when it is a hidden layer's (0 < l < nlayers), else in FP32.
static bool act_bf16(const dirac_ptc *n, int l) { return l > 0 && l < n->nlayers; }
static size_t act_chan_bytes(const dirac_ctx *c, const dirac_ptc *n, int l) {
    return act_bf16(n, l) ? chan_vecs<bf16s>(c->g.vhp) * sizeof(uint4) : chan_vecs<float>(c->g.vhp) * sizeof(float4);
}

void ptc_ensure_acts(dirac_ctx *c, dirac_ptc *n) {
    const size_t chanb = chan_vecs<float>(c->g.vhp) * sizeof(float4);
    size_t need = 0;
    for (int l = 0; l <= n->nlayers; ++l) need += (size_t)n->ch[l] * act_chan_bytes(c, n, l);
    n->acts.alloc(need);
    int maxc = 0;
    for (int l = 0; l <= n->nlayers; ++l) maxc = std::max(maxc, n->ch[l]);
    n->gbuf.alloc(2 * (size_t)maxc * chanb);
    if (n->contract_last()) n->zbuf.alloc((size_t)kPaths * chanb);
    size_t maxpart = 0;  // the weight-gradient slices of the largest layer
    for (int l = 0; l < n->nlayers; ++l)
        maxpart = std::max(maxpart, wgrad_part_bytes(c->g.vhp, n->ch[l], n->ch[l + 1], act_bf16(n, l)));
    n->part.alloc(maxpart);
}

float *ptc_act(dirac_ctx *c, dirac_ptc *n, int l) {
    size_t off = 0;
    for (int k = 0; k < l; ++k) off += (size_t)n->ch[k] * act_chan_bytes(c, n, k);
    return (float *)((char *)n->acts.p + off);
}

// Input and output vectors a caller hands to the network are read and written in place where the kernels can
// (in_place; in: acts[0] otherwise, copied by the caller of these functions).
// forward: the input is `in`, or acts[0] when that is NULL; leaves the output in `out`, or acts[nlayers], and,
// with keep_all, every hidden layer's output in acts[l + 1] (the backward pass needs them).  With eo
// the input's odd half must be zero, and only the even half of the output is formed (a network of
// one layer forms both).
void ptc_forward_acts(dirac_ctx *c, dirac_ptc *n, hipStream_t s, bool keep_all, bool eo, const void *in, void *out) {
    PtcGeom a = geom_of(c, s);
    auto act = [&](int l) -> void * {
        if (l == 0 && in) return const_cast<void *>(in);
        if (l == n->nlayers && out) return out;
        return ptc_act(c, n, l);
    };
    const int L = n->nlayers;
    const bool cf = n->contract_last();
    for (int l = 0; l < (cf ? L - 1 : L); ++l) {
        ZArgs zo;
        if (cf && l == L - 2) {
            zo.Az = (const uint2 *)n->afz.p;
            zo.z = n->zbuf.p;
            zo.store_y = keep_all;
            if (eo) zo.eo |= kEoOut;
        }
        if (eo && l == 0) zo.eo |= kEoIn;
        const Io io = act_bf16(n, l + 1) ? (act_bf16(n, l) ? Io::Mid : Io::In) : Io::F32;
        layer_dispatch(a, n->ch[l], n->ch[l + 1], act(l), (const uint4 *)n->afw.p + n->afw_off[l], act(l + 1), io, s, zo);
    }
    if (cf) {
        const int npar = eo ? 1 : 2;
        k_ptc_tsum<<<(int)((npar * c->vh + 255) / 256), 256, 0, s>>>(a, npar, (const float4 *)n->zbuf.p,
                                                                     (float4 *)act(L));
        HIP_CHECK(hipGetLastError());
    }
}

// backward from g (dL/dy*, FP32 NATIVE full, 1 channel) at the output: accumulates dL/dW* into
// n->grad and, when gin is given, writes dL/dx* of the input (`in`, or acts[0] when that is NULL).
void ptc_backward_acts(dirac_ctx *c, dirac_ptc *n, const void *g_out, void *gin, hipStream_t s, const void *in) {
    PtcGeom a = geom_of(c, s);
    const size_t chanb = chan_vecs<float>(c->g.vhp) * sizeof(float4);
    int maxc = 0;
    for (int l = 0; l <= n->nlayers; ++l) maxc = std::max(maxc, n->ch[l]);
    char *gA = (char *)n->gbuf.p, *gB = gA + (size_t)maxc * chanb;
    const void *g = g_out;  // the gradient at the current layer's output
    if (!in_place(g_out)) {
        HIP_CHECK(hipMemcpyAsync(gA, g_out, (size_t)n->ch[n->nlayers] * chanb, hipMemcpyDeviceToDevice, s));
        g = gA;
    }
    for (int l = n->nlayers - 1; l >= 0; --l) {
        const int nin = n->ch[l], nout = n->ch[l + 1];
        const int nw = (int)ptc_nweights(n, l);
        wgrad_dispatch(a, nin, nout, l == 0 && in ? in : ptc_act(c, n, l), act_bf16(n, l), g, n->part.p,
                       (float2 *)n->grad.p + n->off[l], s);
        if (l == 0 && !gin) break;
        k_adjoint_weights<<<(nw + 255) / 256, 256, 0, s>>>(nout, nin, (const uint32_t *)n->wbf.p + n->off[l],
                                                           (uint32_t *)n->wt.p + n->off[l]);
        HIP_CHECK(hipGetLastError());
        uint4 *afb = (uint4 *)n->afb.p + n->afb_off[l];
        build_afrags(nout, nin, (const uint32_t *)n->wt.p + n->off[l], afb, s);
        void *dst = l == 0 ? gin : (void *)gB;
        layer_dispatch(a, nout, nin, g, afb, dst, Io::F32, s);
        std::swap(gA, gB);
        g = gA;
    }
}

void ptc_adam(dirac_ptc *n, double lr, hipStream_t s) {
    n->step += 1;
    // the decay rates and the bias corrections 1 - b^t in FP64, each rounded to FP32 once
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    const double c1 = 1.0 - std::pow(b1, (double)n->step), c2 = 1.0 - std::pow(b2, (double)n->step);
    const int nr = (int)(2 * n->total);
    k_adam<<<(nr + 255) / 256, 256, 0, s>>>(nr, (float *)n->w.p, (const float *)n->grad.p, (float *)n->m.p,
                                           (float *)n->v.p, (uint16_t *)n->wbf.p, (float)lr, (float)b1,
                                           (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)eps, (float)c1,
                                           (float)c2);
    HIP_CHECK(hipGetLastError());
    refresh_afrags(n, s);
}

}  // namespace dl
