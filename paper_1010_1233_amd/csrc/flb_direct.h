// flb_direct.h -- line transforms by direct sums.
#pragma once

#include "flb_internal.h"

namespace flbdev {

// Line transforms by direct sums, for short lines of any length.  A task adds
// up cosine and sine sums over j < n / 2 of the folded values z_j + z_{n-j}
// and z_j - z_{n-j}; for even n the even and the odd j apart, as
// exp(-2 pi i j (n/2 - k) / n) is (-1)^j times the conjugate of that of k.
// So one pass over a line gives the outputs k, n - k, n/2 - k and n/2 + k,
// about n operations an output, in two barriers whatever the length, where
// Bluestein's convolution takes two transforms of two to four times the
// length.  LDS bounds it: one root and two values per pass and step.
__device__ __forceinline__ float2 operator+(float2 a, float2 b)
{
    return make_float2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ float2 operator-(float2 a, float2 b)
{
    return make_float2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ float fma_z(float w, float z, float a) { return fmaf(w, z, a); }
__device__ __forceinline__ float2 fma_z(float w, float2 z, float2 a)
{
    return make_float2(fmaf(w, z.x, a.x), fmaf(w, z.y, a.y));
}

// The sums of NF lines of real (float) or complex (float2) values at output
// k: line f's value j is z(f, j); c[f][p], s[f][p]: over the j of parity p
// (all in c[f][0], s[f][0] for odd n).
template <int NF, typename Z, typename F>
__device__ __forceinline__ void direct_sums(int n, int k, const float2 *roots, F &&z,
                                            Z (&c)[NF][2], Z (&s)[NF][2])
{
    const bool even = (n & 1) == 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        c[f][0] = z(f, 0);
        c[f][1] = s[f][0] = s[f][1] = Z{};
    }
    auto term = [&](int j, int m, int p) {
        const float2 w = roots[m];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const Z a = z(f, j), b = z(f, n - j);
            c[f][p] = fma_z(w.x, a + b, c[f][p]);
            s[f][p] = fma_z(w.y, a - b, s[f][p]);
        }
    };
    const int last = (n - 1) / 2;  // the j below n / 2
    int m = 0;
    auto next = [&]() {
        m += k;
        m = m >= n ? m - n : m;
        return m;
    };
    if (even) {
        int j = 1;
        for (; j + 1 <= last; j += 2) {
            const int m1 = next(), m2 = next();
            term(j, m1, 1);
            term(j + 1, m2, 0);
        }
        if (j <= last) term(j, next(), 1);
        // j = n / 2: (-1)^k
        const float w = (k & 1) ? -1.f : 1.f;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const Z v = z(f, n / 2);
            if ((n / 2) & 1) c[f][1] = fma_z(w, v, c[f][1]);
            else c[f][0] = fma_z(w, v, c[f][0]);
        }
    } else {
        for (int j = 1; j <= last; ++j) term(j, next(), 0);
    }
}
// Tasks per line: k = 0 .. n/4 for even n, 0 .. n/2 for odd.
__host__ __device__ inline int direct_tasks(int n) { return ((n & 1) ? n / 2 : n / 4) + 1; }

// The outputs of a complex line from its sums: emit(ky, values of the NF
// lines), each ky once.
template <int NF, typename F>
__device__ __forceinline__ void direct_outputs(int n, int k, const float2 (&c)[NF][2],
                                               const float2 (&s)[NF][2], F &&emit)
{
    // cosine sums C and sine sums S (of -sin): output C + i S at k, C - i S
    // at n - k
    auto both = [&](int ky, float sg) {
        float2 C[NF], S[NF], X[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            C[f] = fma_z(sg, c[f][1], c[f][0]);
            S[f] = fma_z(sg, s[f][0], s[f][1]);  // sg = 1: the sum; -1: odd less even
            X[f] = make_float2(C[f].x - S[f].y, C[f].y + S[f].x);
        }
        emit(ky, X);
        if (ky == 0 || 2 * ky == n) return;
#pragma unroll
        for (int f = 0; f < NF; ++f) X[f] = make_float2(C[f].x + S[f].y, C[f].y - S[f].x);
        emit(n - ky, X);
    };
    both(k, 1.f);
    if ((n & 1) == 0 && 4 * k != n) both(n / 2 - k, -1.f);
}

}  // namespace flbdev
