// flb_collide.h -- one site's update (relaxation, noise) as every kernel
// that steps a D2Q9 lattice inlines it: the same bits in all of them.
#pragma once

#include "flb_device.h"

namespace flbdev {

// Eq. (5) for one site on deviations d_i = f_i - w_i rho0, in place.
// Moments are kept in a scaled basis so the back transform has unit
// coefficients: s3 = 3/2 M^3, s4 = 3 M^4, s5 = M^5, s6 = sqrt(3/2) M^6,
// s7 = sqrt(3/2) M^7, s8 = M^8; M^1 = sqrt(3) jx, M^2 = sqrt(3) jy.  The
// deviation from w_i rho0 shifts only M^0 (sum_i w_i m_i^a = 0 for a > 0).
// Only the change of moments 3..8, -(M^a - M^{a,0})/tau^a + xi^a, is
// transformed back and added to the gathered values: density and momentum
// ride along untouched, so FP32 weights such as 1/9 (not exact in binary)
// cannot bias them step after step; what remains is zero-mean rounding.
template <bool NOISE>
__device__ __forceinline__ void collide(float (&d)[9], const LatticeParams &P, const float (&z)[6])
{
    // only the written fmaf calls fuse: a multiply and an add are never
    // contracted by the compiler, whose choice could differ between the
    // kernels that inline this (their results must be the same bits)
#pragma clang fp contract(off)
    const float a = d[1] + d[3], b = d[2] + d[4];
    const float c = d[5] + d[7], e = d[6] + d[8];
    const float ab = a + b, ce = c + e;
    const float drho = d[0] + ab + ce;
    const float x13 = d[1] - d[3], y24 = d[2] - d[4];
    const float p57 = d[5] - d[7], p68 = d[6] - d[8];
    const float q68 = p57 - p68, r68 = p57 + p68;  // shared with g6, g7
    const float jx = x13 + q68;
    const float jy = y24 + r68;

    // In the scaled basis s3 = 9/4 (a - b), s4 = 9 (c - e), s5, s6 = 3/2 g6,
    // s7 = 3/2 g7, s8, and Eq. (10): e3 = 9/4 (jx^2 - jy^2)/rho,
    // e4 = 9 jx jy/rho, e5 = 3/2 (jx^2 + jy^2)/rho, the others 0.  The
    // constant factors ride in per-lattice coefficients (fcoef): t3 =
    // 9/4 omega3 ((jx^2 - jy^2)/rho - (a - b)), t4 = 9 omega4 (jx jy/rho -
    // (c - e)), and the ghost changes are kept doubled, u6 = 2 t6 =
    // -3 omega6 g6 (+ 2 amp z), u7 = 2 t7 likewise.
    const float s5 = fmaf(0.5f, ab, fmaf(2.0f, ce, -d[0]));
    const float g6 = fmaf(2.0f, q68, -x13);
    const float g7 = fmaf(2.0f, r68, -y24);
    const float s8 = fmaf(0.5f, d[0], fmaf(2.0f, ce, -ab));
    const float ir = __builtin_amdgcn_rcpf(P.rho0 + drho);
    const float jyy = jy * jy;

    // change of each scaled moment, Eq. (5) and Eq. (8)
    float t3 = P.fcoef[0] * fmaf(fmaf(jx, jx, -jyy), ir, -(a - b));
    float t4 = P.fcoef[1] * fmaf(jx * jy, ir, -(c - e));
    float t5 = P.omega[2] * fmaf(1.5f * fmaf(jx, jx, jyy), ir, -s5);
    float u6 = P.fcoef[2] * g6;
    float u7 = P.fcoef[3] * g7;
    float t8 = -P.omega[5] * s8;
    if constexpr (NOISE) {
        t3 = fmaf(P.amp[0], z[0], t3);
        t4 = fmaf(P.amp[1], z[1], t4);
        t5 = fmaf(P.amp[2], z[2], t5);
        u6 = fmaf(P.fcoef[4], z[3], u6);
        u7 = fmaf(P.fcoef[5], z[4], u7);
        t8 = fmaf(P.amp[5], z[5], t8);
    }

    // d*_i = d_i + w_i sum_{a>=3} m_i^a dM^a
    const float A = fmaf(0.5f, t5, -t8);
    const float B = 2.0f * (t5 + t8);
    const float PpQ = u6 + u7, PmQ = u6 - u7;  // 2 t6 +- 2 t7
    const float Ap = A + t3, Am = A - t3;
    constexpr float w0 = 4.0f / 9.0f, w1 = 1.0f / 9.0f, w5 = 1.0f / 36.0f;
    d[0] = fmaf(w0, fmaf(0.5f, t8, -t5), d[0]);
    d[1] = fmaf(w1, fmaf(-0.5f, u6, Ap), d[1]);
    d[3] = fmaf(w1, fmaf(0.5f, u6, Ap), d[3]);
    d[2] = fmaf(w1, fmaf(-0.5f, u7, Am), d[2]);
    d[4] = fmaf(w1, fmaf(0.5f, u7, Am), d[4]);
    d[5] = fmaf(w5, (B + t4) + PpQ, d[5]);
    d[6] = fmaf(w5, (B - t4) - PmQ, d[6]);
    d[7] = fmaf(w5, (B + t4) - PpQ, d[7]);
    d[8] = fmaf(w5, (B - t4) + PmQ, d[8]);
}

// The same collision for the 16-bit formats, on the stored scaled
// deviations q_i = (d_i - F_i) / s_i themselves (F the deviation of the
// reference state f^0(rho0, u0), s_i = sqrt(mu rho0 w_i) one scale per
// velocity class): every moment above is a linear function of the d_i, so
// it is the class-scaled sum of the q_i plus the moment of F, and the
// change of d_i, w_i sum_a m_i^a dM^a, is a change of q_i by w_i / s_i times
// that sum.  No value is decoded to d or encoded back one by one.
template <bool NOISE>
__device__ __forceinline__ void collide_q(float (&q)[9], const LatticeParams &P,
                                          const float (&z)[6])
{
#pragma clang fp contract(off)  // as in collide
    const float *C = P.qcoef, *K = P.qoff;
    const float qa = q[1] + q[3], qb = q[2] + q[4];
    const float qc = q[5] + q[7], qe = q[6] + q[8];
    const float qab = qa + qb, qce = qc + qe;
    const float qx = q[1] - q[3], qy = q[2] - q[4];
    const float qp = q[5] - q[7], qm = q[6] - q[8];
    const float pmm = qp - qm, ppm = qp + qm;
    // C: s0, s1, s5, 9/4 s1, 9 s5, s1/2, 2 s5, 3 s5, 3/2 s1, s0/2
    const float drho = fmaf(C[0], q[0], fmaf(C[1], qab, fmaf(C[2], qce, K[0])));
    const float jx = fmaf(C[1], qx, fmaf(C[2], pmm, K[1]));
    const float jy = fmaf(C[1], qy, fmaf(C[2], ppm, K[2]));
    const float s3 = fmaf(C[3], qa - qb, K[3]);
    const float s4 = fmaf(C[4], qc - qe, K[4]);
    const float s5 = fmaf(C[5], qab, fmaf(C[6], qce, fmaf(-C[0], q[0], K[5])));
    const float s6 = fmaf(C[7], pmm, fmaf(-C[8], qx, K[6]));
    const float s7 = fmaf(C[7], ppm, fmaf(-C[8], qy, K[7]));
    const float s8 = fmaf(C[9], q[0], fmaf(C[6], qce, fmaf(-C[1], qab, K[8])));

    // Eq. (10), relaxation and noise exactly as in collide()
    const float ir = __builtin_amdgcn_rcpf(P.rho0 + drho);
    const float jxx = jx * jx, jyy = jy * jy;
    const float e3 = 2.25f * (jxx - jyy) * ir;
    const float e4 = 9.0f * (jx * jy) * ir;
    const float e5 = 1.5f * (jxx + jyy) * ir;
    float t3 = P.omega[0] * (e3 - s3);
    float t4 = P.omega[1] * (e4 - s4);
    float t5 = P.omega[2] * (e5 - s5);
    float t6 = -P.omega[3] * s6;
    float t7 = -P.omega[4] * s7;
    float t8 = -P.omega[5] * s8;
    if constexpr (NOISE) {
        t3 = fmaf(P.amp[0], z[0], t3);
        t4 = fmaf(P.amp[1], z[1], t4);
        t5 = fmaf(P.amp[2], z[2], t5);
        t6 = fmaf(P.amp[3], z[3], t6);
        t7 = fmaf(P.amp[4], z[4], t7);
        t8 = fmaf(P.amp[5], z[5], t8);
    }
    // q*_i = q_i + (w_i / s_i) sum_{a>=3} m_i^a dM^a
    const float A = fmaf(0.5f, t5, -t8);
    const float B = 2.0f * (t5 + t8);
    const float P6 = 2.0f * t6, Q7 = 2.0f * t7;
    const float w0 = P.qback[0], w1 = P.qback[1], w5 = P.qback[2];
    q[0] = fmaf(w0, fmaf(0.5f, t8, -t5), q[0]);
    q[1] = fmaf(w1, (A + t3) - t6, q[1]);
    q[3] = fmaf(w1, (A + t3) + t6, q[3]);
    q[2] = fmaf(w1, (A - t3) - t7, q[2]);
    q[4] = fmaf(w1, (A - t3) + t7, q[4]);
    q[5] = fmaf(w5, (B + t4) + (P6 + Q7), q[5]);
    q[6] = fmaf(w5, (B - t4) - (P6 - Q7), q[6]);
    q[7] = fmaf(w5, (B + t4) - (P6 + Q7), q[7]);
    q[8] = fmaf(w5, (B - t4) + (P6 - Q7), q[8]);
}

// The step kernels' working value of a stored population: the FP32
// deviation itself, or for the 16-bit formats the stored scaled deviation
// (collide_q works on it); `out` rounds a working value to the storage
// format (materialised in FP32 first: see round_point).
template <int S> struct Work {
    using T = typename Codec<S>::T;
    static __device__ __forceinline__ float in(T v) { return (float)v; }
    static __device__ __forceinline__ T out(float x)
    {
        if constexpr (S == kF32) return x;
        else return (T)round_point(x);
    }
};

// Collision of one site, including its noise draw, on working values
// (Work<S>).
template <bool NOISE, int S>
__device__ __forceinline__ void update_site(float (&d)[9], const LatticeParams &P, uint32_t site,
                                            uint32_t t, uint32_t key0, uint32_t key1)
{
    float z[6] = {0, 0, 0, 0, 0, 0};
    if constexpr (NOISE) normals6(philox4x32_10(make_uint4(site, t, P.stream_id, 0u), key0, key1), z);
    if constexpr (S == kF32) collide<NOISE>(d, P, z);
    else collide_q<NOISE>(d, P, z);
}

// a working value as the next level reads it back from storage
template <int S> __device__ __forceinline__ float stored(float x)
{
    if constexpr (S == kF32) return x;
    else return Work<S>::in(Work<S>::out(x));
}

}  // namespace flbdev
