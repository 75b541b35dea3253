// sigma without branches, for code that evaluates it for many elements at once; td_act and td_act_f64 (common.h) are the same functions
// through the math library.
#pragma once
#include "common.h"

// sigma in the epilogues, where it is evaluated for whole rows of accumulators: no branches, so that several elements are under
// way at once.  GELU = z Phi(z): for |z| < 1 Phi = 1/2 + z S(z^2), else from Phi(-|z|) = t exp(P(t) - z^2 / 2), t = 1 / (1 + 0.4 |z|);
// S and P are minimax fits (to 3e-10 and 3e-8) of the two functions so defined.  Root mean square error against 64 bits for z from
// N(0, 1.6^2), measured here and for the library functions' form (td_act): 3.48e-8 and 3.99e-8, with tanh 3.46e-8 and 3.93e-8; from
// other spreads (0.5 to 8) no larger than the latter's either, and below -2 a tenth of it, which cancels there.
// Infinities and NaNs give what they gave: +inf, and NaN for -inf.
template <int ACT> __device__ __forceinline__ float act_flat(float z) {
    if constexpr (ACT == TARDIS_ACT_GELU_ERF) {
        const float u = fabsf(z), w = z * z;
        const float t = __builtin_amdgcn_rcpf(fmaf(0.4f, u, 1.0f));
        float s = -7.6011511e-06f, p = -0.43888903f;
        s = fmaf(s, w, 1.13367088e-04f);
        s = fmaf(s, w, -1.18623779e-03f);
        s = fmaf(s, w, 9.97329503e-03f);
        s = fmaf(s, w, -6.64903596e-02f);
        s = fmaf(s, w, 0.398942292f);
        p = fmaf(p, t, 1.36559796f);                        // (P and z^2 / 2 in units of log 2)
        p = fmaf(p, t, -1.33750927f);
        p = fmaf(p, t, 0.194332317f);
        p = fmaf(p, t, -0.0835891962f);
        p = fmaf(p, t, 0.504601836f);
        p = fmaf(p, t, 1.44168389f);
        p = fmaf(p, t, -2.64764786f);
        const float q = t * __builtin_amdgcn_exp2f(fmaf(u * -0.721347520f, u, p));
        return z * (u < 1.0f ? fmaf(z, s, 0.5f) : z > 0.0f ? 1.0f - q : q);
    } else if constexpr (ACT == TARDIS_ACT_GELU_TANH) {
        // (1 + tanh v) / 2 = 1 - q, of -v q, with q = e / (1 + e) and e = exp(-2 |v|) <= 1 (in units of log 2): what the exponential and
        // the reciprocal round is no part of the sum that way
        const float u = fabsf(z);
        const float e = __builtin_amdgcn_exp2f(-u * fmaf(0.102943240f * z, z, 2.30220819f));
        const float q = e * __builtin_amdgcn_rcpf(1.0f + e);
        return z * (z > 0.0f ? 1.0f - q : q);
    } else {
        return td_act(z, ACT);
    }
}

// sigma in fp64 without branches, for the calibration's samples.  GELU = z Phi(z) from Phi(-|z|) = erfc(x) / 2, x = |z| / sqrt(2):
// (1 + 2 x) exp(x^2) erfc(x) is a polynomial in (x - K) / (x + K) (the substitution of Shepherd and Laframboise, Math. Comp. 36,
// 1981; K = 3.75, degree 20, the coefficients interpolate it at 400 Chebyshev points).  Against the library's erf (two
// branches, of which a wavefront takes both): root mean square error 8.5e-17 instead of 1.6e-16 for z from -8 to 8, largest 8.9e-16 on either side.
__device__ __forceinline__ double rcp_f64(double a) {              // a: a normal number
    double r = __builtin_amdgcn_rcp(a);
    r = fma(fma(-a, r, 1.0), r, r);
    return fma(fma(-a, r, 1.0), r, r);
}
__device__ __forceinline__ double exp_f64(double y) {              // |y| <= 2^20: Taylor's series, 13 terms, on |r| <= log(2) / 2
    const double n = rint(y * 1.4426950408889634074);
    constexpr double kHead = 0.6931471796706319, kRest = 8.893134238886677e-10;   // log(2): its first 30 bits, so that n times them is exact; the rest
    const double r = fma(n, -kRest, fma(n, -kHead, y));
    constexpr double c[13] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
                              1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600};
    double s = c[12];
#pragma unroll
    for (int k = 11; k >= 0; --k) s = fma(s, r, c[k]);
    return ldexp(s, (int)n);
}
template <int ACT> __device__ __forceinline__ double act_flat_f64(double z) {
    if constexpr (ACT == TARDIS_ACT_GELU_ERF) {
        constexpr double K = 3.75;
        constexpr double c[21] = {
            1.2375126308378264, -0.14024059858550675, 0.0035854154857959016,
            0.08227673848715551, -0.10880393015501522, 0.09230432122566992,
            -0.05869339838179839, 0.028362276763635674, -0.009746581233908157,
            0.001755629481119746, 0.00029372158155062665, -0.0002901662170030672,
            5.162565962208987e-05, 2.2409881005582833e-05, -1.1399206978826016e-05,
            -1.0082073330153207e-06, 1.6955385768824271e-06, -2.78242458762179e-08,
            -2.1408381400078725e-07, 8.543261174054351e-09, 1.7505899450043215e-08};
        const double x = fmin(fabs(z) * 0.70710678118654752440, 40.0);     // (erfc(40) is 0, and infinities stay what they were)
        const double p = x + K, w = fma(2.0, x, 1.0), r = rcp_f64(p * w);
        const double t = (x - K) * (w * r);
        double s = c[20];
#pragma unroll
        for (int k = 19; k >= 0; --k) s = fma(s, t, c[k]);
        const double half = 0.5 * s * (p * r) * exp_f64(-x * x);
        return z * (z > 0.0 ? 1.0 - half : half);
    } else if constexpr (ACT == TARDIS_ACT_GELU_TANH) {
        // as in 32 bits; |v| beyond 1e5 is 1e5 (where e is 0)
        const double v = 0.79788456080286535588 * (z + 0.044715 * z * z * z);
        const double e = exp_f64(fmax(-2.0 * fabs(v), -1e5));
        const double q = e * rcp_f64(1.0 + e);
        return z * (z > 0.0 ? 1.0 - q : q);
    } else {
        return td_act_f64(z, ACT);
    }
}
