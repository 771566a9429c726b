// Device arithmetic of the CG scalars (slots in blas.h), shared by the kernel
// that sums partials (finalize) and by the kernels that sum few of them where
// the result is used.
#pragma once

#include <hip/hip_runtime.h>

#include "blas.h"

namespace dwf {

__device__ __forceinline__ double cg_alpha(double rr, double qq) {
    return (qq > 0.0 && isfinite(qq)) ? rr / qq : 0.0;
}
__device__ __forceinline__ double cg_beta(double rr_new, double rr) { return rr > 0.0 ? rr_new / rr : 0.0; }

// Sum of n <= CG_FEW partials in every lane of a wave, in two steps so that
// other loads can be issued in between.  The bits are those of finalize_kernel's
// sum: 64 partials by a butterfly, then the sums of the groups by another; absent
// ones are zeros there too.
constexpr int CG_FEW = 256;
__device__ __forceinline__ void load_few(const double* p, int n, double (&v)[CG_FEW / 64]) {
#pragma unroll
    for (int k = 0; k < CG_FEW / 64; ++k) {
        const int i = k * 64 + ((int)threadIdx.x & 63);
        v[k] = i < n ? p[i] : 0.0;
    }
}
__device__ __forceinline__ double sum_few(double (&v)[CG_FEW / 64]) {
    double w = 0.0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int k = 0; k < CG_FEW / 64; ++k) v[k] += __shfl_xor(v[k], off, 64);
#pragma unroll
    for (int k = 0; k < CG_FEW / 64; ++k)
        if (((int)threadIdx.x & 63) == k) w = v[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) w += __shfl_xor(w, off, 64);
    return w;
}

// alpha = RR / QQ from the partials of QQ (load_few).  `first` (one thread of the
// launch) stores the step's scalars; RR itself is only read here.
__device__ __forceinline__ double alpha_of_partials(double (&v)[CG_FEW / 64], double* scal, double* alpha_copy,
                                                    bool first) {
    const double rr = scal[CG_RR], qq = sum_few(v), a = cg_alpha(rr, qq);
    if (first) {
        if (!isfinite(qq)) scal[CG_NANFLAG] = 1.0;
        scal[CG_QQ] = qq;
        scal[CG_ALPHA] = a;
        scal[CG_RROLD] = rr;
        if (alpha_copy) *alpha_copy = a;
    }
    return a;
}

// beta = RR_new / RR_old from the partials of RR_new; RR_old is only read here
__device__ __forceinline__ double beta_of(const CgBeta& b) {
    if (!b.sum) return *b.beta;
    double v[CG_FEW / 64];
    load_few(b.sum, b.nsum, v);
    const double old = b.scal[CG_RROLD], rr = sum_few(v), be = cg_beta(rr, old);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const bool bad = !isfinite(rr) || b.scal[CG_NANFLAG] != 0.0;
        if (bad) b.scal[CG_NANFLAG] = 1.0;
        b.scal[CG_RRNEW] = rr;
        b.scal[CG_BETA] = be;
        b.scal[CG_RR] = rr;
        if (b.host) {
            b.host[CG_RR] = rr;
            b.host[CG_NANFLAG] = bad ? 1.0 : 0.0;
        }
    }
    return be;
}

}  // namespace dwf
