// Entry points of the per-precision hop translation units (hop_f64.hip ... hop_bf16.hip):
// hop_t<S> of hop_kernels.h with S the storage type of the precision.
#pragma once

#include "internal.h"

namespace dl {

// hop_t<S> of hop_kernels.h for one storage precision, one translation unit each
void hop_prec_f64(dirac_ctx *c, void *out, const void *in, const void *chi, int p, HopMode mode, double coef,
                  int dagger, hipStream_t s, int nrhs, const int *active, bool no_tune);
void hop_prec_f32(dirac_ctx *c, void *out, const void *in, const void *chi, int p, HopMode mode, double coef,
                  int dagger, hipStream_t s, int nrhs, const int *active, bool no_tune);
void hop_prec_f16(dirac_ctx *c, void *out, const void *in, const void *chi, int p, HopMode mode, double coef,
                  int dagger, hipStream_t s, int nrhs, const int *active, bool no_tune);
void hop_prec_bf16(dirac_ctx *c, void *out, const void *in, const void *chi, int p, HopMode mode, double coef,
                   int dagger, hipStream_t s, int nrhs, const int *active, bool no_tune);

// One launch of the direction-parallel kernel: out_p = mode(coef H in_{1-p}) for the parities p .. p + np - 1,
// vectors in the layouts given (dirac_layout; half: of one parity, else full vectors).  HOP_INV or HOP_CLOV.
struct HopDirCall {
    void *out;
    const void *in, *chi;
    int in_lay, chi_lay, out_lay, half, p, np;
    HopMode mode;
    double coef;
    int dagger;
    dirac_prec pr;
};
void hop_dir_f64(dirac_ctx *c, const HopDirCall &k, hipStream_t s);
void hop_dir_f32(dirac_ctx *c, const HopDirCall &k, hipStream_t s);
void hop_dir_f16(dirac_ctx *c, const HopDirCall &k, hipStream_t s);
void hop_dir_bf16(dirac_ctx *c, const HopDirCall &k, hipStream_t s);

}  // namespace dl
