// Hopping term between parities, fused with the clover field, and the even-odd Schur and full
// operators built from it.  The kernels and their launch shapes are in hop_kernels.h, compiled
// once per storage precision (hop_f64.hip, hop_f32.hip, hop_f16.hip, hop_bf16.hip).
#include <cstdlib>

#include "hop_launch.h"
#include "internal.h"

namespace dl {

void hop_apply(dirac_ctx *c, void *out, const void *in, const void *chi, int p, HopMode mode, double coef, int dagger,
               dirac_prec pr, hipStream_t s, int nrhs, const int *active, bool no_alloc) {
    require(nrhs >= 1, "nrhs must be positive");
    require(p == 0 || p == 1, "parity must be 0 (even) or 1 (odd)");
    PrecFields &f = c->f[pr];
    if (no_alloc)
        require(f.links_ready && (mode == HOP_PLAIN || f.clover_ready),
                std::string("the ") + prec_name(pr) + " fields have not been built; any apply in this precision builds them");
    else
        ensure_prec(c, pr, s);
    require(mode != HOP_INV || f.inv_ready[p], "clover inverse of this parity not computed; call clover_invert");
    switch (pr) {
        case DIRAC_F64: hop_prec_f64(c, out, in, chi, p, mode, coef, dagger, s, nrhs, active, no_alloc); break;
        case DIRAC_F32: hop_prec_f32(c, out, in, chi, p, mode, coef, dagger, s, nrhs, active, no_alloc); break;
        case DIRAC_F16: hop_prec_f16(c, out, in, chi, p, mode, coef, dagger, s, nrhs, active, no_alloc); break;
        case DIRAC_BF16: hop_prec_bf16(c, out, in, chi, p, mode, coef, dagger, s, nrhs, active, no_alloc); break;
        default: throw Error(DIRAC_EINVAL, "unknown precision");
    }
}

// D-hat in_e = A_ee in_e - D_eo A_oo^-1 D_oe in_e, D_eo = -H_eo / 2:
//   t_o = A_oo^-1 (-1/2 H_oe in_e);   out_e = A_ee in_e + 1/2 H_eo t_o
void schur_apply(dirac_ctx *c, void *out_e, const void *in_e, int dagger, dirac_prec pr, hipStream_t s, int nrhs,
                 const int *active) {
    ensure_prec(c, pr, s);
    PrecFields &f = c->f[pr];
    require(f.inv_ready[1], "odd-site clover inverse not available (clover_invert failed or was not run)");
    f.tmp_half.alloc((size_t)nrhs * 24 * real_size(pr) * c->g.vhp);
    schur_apply_into(c, out_e, in_e, f.tmp_half.p, dagger, pr, s, nrhs, active, false);
}

// The two launches of D-hat with the odd intermediate t_o in `tmp` (nrhs odd half vectors of pr);
// no_alloc: build nothing and time nothing (the fields of pr must exist).
void schur_apply_into(dirac_ctx *c, void *out_e, const void *in_e, void *tmp, int dagger, dirac_prec pr,
                      hipStream_t s, int nrhs, const int *active, bool no_alloc) {
    require(c->f[pr].inv_ready[1], "odd-site clover inverse not available (clover_invert failed or was not run)");
    hop_apply(c, tmp, in_e, nullptr, 1, HOP_INV, -0.5, dagger, pr, s, nrhs, active, no_alloc);
    hop_apply(c, out_e, tmp, in_e, 0, HOP_CLOV, 0.5, dagger, pr, s, nrhs, active, no_alloc);
}

// D in: out_p = A_pp in_p - 1/2 H in_{1-p} for both parities (NATIVE full vectors).
void full_apply(dirac_ctx *c, void *out, const void *in, int dagger, dirac_prec pr, hipStream_t s) {
    const size_t hb = (size_t)24 * real_size(pr) * c->g.vhp;
    const char *ie = (const char *)in, *io = ie + hb;
    char *oe = (char *)out, *oo = oe + hb;
    hop_apply(c, oe, io, ie, 0, HOP_CLOV, -0.5, dagger, pr, s);
    hop_apply(c, oo, ie, io, 1, HOP_CLOV, -0.5, dagger, pr, s);
}

namespace {
void hop_dir(dirac_ctx *c, const HopDirCall &k, hipStream_t s) {
    switch (k.pr) {
        case DIRAC_F64: hop_dir_f64(c, k, s); break;
        case DIRAC_F32: hop_dir_f32(c, k, s); break;
        case DIRAC_F16: hop_dir_f16(c, k, s); break;
        case DIRAC_BF16: hop_dir_bf16(c, k, s); break;
        default: throw Error(DIRAC_EINVAL, "unknown precision");
    }
}
bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
}  // namespace

// Operators on vectors in the caller's layout without conversion passes: the direction-parallel kernel reads and
// writes them as they are.  Taken for lattices of at most kDirSites sites per parity and 16-byte aligned vectors
// (it loads 16 bytes at a time); on large ones its reads of the caller's sites, 192 or 96 bytes apart, touch a cache
// line each and a conversion is faster.  Direct against converted, calls queued one after another: D on a LEX vector in FP64
// 12^4 19 against 42 us, 16 x 8 x 16^2 (16,384 sites) 20 against 49, 14 x 18 x 12 x 16 (24,192) 32 against 40, 16^4 40 against
// 44, 16^3 x 24 (49,152) 59 against 55; the Schur operator on an EO vector 16 against 32, 19 against 34, 31 against 37, 33
// against 41, 48 against 49.  The line lies below the crossing, where direct calls are faster by half or more in every layout.
// A launch shape forced by DIRAC_HOP_SHAPE is one of the NATIVE kernels', so then every call is converted.
constexpr int kDirSites = 16384;

bool direct_layout(const dirac_ctx *c, const void *out, const void *in) {
    return c->g.vh <= kDirSites && aligned16(out) && aligned16(in) && !getenv("DIRAC_HOP_SHAPE");
}

void schur_apply_direct(dirac_ctx *c, void *out_e, const void *in_e, dirac_layout lay, int dagger, dirac_prec pr,
                        hipStream_t s) {
    ensure_prec(c, pr, s);
    PrecFields &f = c->f[pr];
    require(f.inv_ready[1], "odd-site clover inverse not available (clover_invert failed or was not run)");
    f.tmp_half.alloc((size_t)24 * real_size(pr) * c->g.vhp);
    const int nat = DIRAC_LAYOUT_NATIVE;
    hop_dir(c, {f.tmp_half.p, in_e, nullptr, lay, nat, nat, 1, 1, 1, HOP_INV, -0.5, dagger, pr}, s);
    hop_dir(c, {out_e, f.tmp_half.p, in_e, nat, lay, lay, 1, 0, 1, HOP_CLOV, 0.5, dagger, pr}, s);
}

// both parities in one launch
void full_apply_direct(dirac_ctx *c, void *out, const void *in, dirac_layout lay, int dagger, dirac_prec pr,
                       hipStream_t s) {
    ensure_prec(c, pr, s);
    hop_dir(c, {out, in, in, lay, lay, lay, 0, 0, 2, HOP_CLOV, -0.5, dagger, pr}, s);
}

}  // namespace dl
