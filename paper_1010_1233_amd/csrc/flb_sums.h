// flb_sums.h -- what every sample kernel computes alike: a site's moments,
// and the FP64 products of one sample's spectra at one k and their addition
// to the correlator sums (Eqs. 11-12).
#pragma once

#include "flb_device.h"

namespace flbdev {

// Non-conserved moments M^3..M^8 (rows of Eq. 9) of a site's deviations.
// The rows are orthogonal to M^0 under the weights, so the moments of the
// deviations are the moments themselves.
__device__ __forceinline__ void moments_of(const float (&d)[9], float (&M)[6])
{
    const float axis = (d[1] + d[3]) + (d[2] + d[4]);
    const float diag = (d[5] + d[7]) + (d[6] + d[8]);
    const float s32 = 1.2247448713915890f, s6 = 2.4494897427831781f;
    M[0] = 1.5f * ((d[1] + d[3]) - (d[2] + d[4]));
    M[1] = 3.0f * ((d[5] + d[7]) - (d[6] + d[8]));
    M[2] = fmaf(0.5f, axis, fmaf(2.0f, diag, -d[0]));
    M[3] = fmaf(s32, d[3] - d[1], s6 * ((d[5] - d[7]) + (d[8] - d[6])));
    M[4] = fmaf(s32, d[4] - d[2], s6 * ((d[5] - d[7]) + (d[6] - d[8])));
    M[5] = fmaf(0.5f, d[0], fmaf(2.0f, diag, -axis));
}

// Fifteen products of the five spectra at one k, in FP64.
__device__ __forceinline__ void products_k(double (&val)[kKinds], const float2 (&X)[5])
{
    double re[5], im[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        re[f] = X[f].x;
        im[f] = X[f].y;
    }
    // a b* = (ar br + ai bi) + i (ai br - ar bi)
#define FLB_RE(u, v) (re[u] * re[v] + im[u] * im[v])
#define FLB_IM(u, v) (im[u] * re[v] - re[u] * im[v])
    const double p[kKinds] = {FLB_RE(0, 0), FLB_RE(1, 1), FLB_RE(2, 2), FLB_RE(3, 3),
                              FLB_RE(4, 4), FLB_RE(3, 4), FLB_IM(3, 4), FLB_RE(0, 1),
                              FLB_IM(0, 1), FLB_RE(0, 2), FLB_IM(0, 2), FLB_RE(0, 3),
                              FLB_IM(0, 3), FLB_RE(0, 4), FLB_IM(0, 4)};
#undef FLB_RE
#undef FLB_IM
#pragma unroll
    for (int q = 0; q < kKinds; ++q) val[q] = p[q];
}

// One read-modify-write of NK FP64 sums at one k (stride kstride): every
// old value is read before any is written, so the reads are in flight
// together (read and write addresses are the same, so the compiler may not
// reorder a later read before an earlier write on its own).
template <int NK, bool NT = false>
__device__ __forceinline__ void add_to_sums(double *a, int64_t kstride, const double (&u)[NK])
{
    double old[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) old[q] = gload<NT>(&a[q * kstride]);
#pragma unroll
    for (int q = 0; q < NK; ++q) gstore<NT>(&a[q * kstride], old[q] + u[q]);
}

// Adds the products of one sample at one k to the sums.
__device__ __forceinline__ void accumulate_k(double *a, int64_t kstride, const float2 (&X)[5])
{
    double val[kKinds];
    products_k(val, X);
    add_to_sums(a, kstride, val);
}

// Squared moduli of the six moment spectra at one k.
__device__ __forceinline__ void moment_products_k(double (&u)[6], const float2 (&X)[6])
{
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const double re = X[f].x, im = X[f].y;
        u[f] = re * re + im * im;
    }
}

// The same, added to kinds kKinds .. kKinds + 5.
__device__ __forceinline__ void accumulate_moments_k(double *a, int64_t kstride,
                                                     const float2 (&X)[6])
{
    double u[6];
    moment_products_k(u, X);
    add_to_sums<6>(a + kKinds * kstride, kstride, u);
}

}  // namespace flbdev
