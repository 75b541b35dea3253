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

// sigma in fp64 without divergent branches, for the calibration's samples.  GELU = z Phi(z): for |z| < 1 Phi = 1/2 + z S(z^2), S interpolated at
// Chebyshev points, else from Phi(-|z|) = erfc(x) / 2, x = |z| / sqrt(2): with p = x - sqrt(1/2) + K, p exp(x^2) erfc(x) is a polynomial in
// 1 - 2 K / p (after the substitution of Shepherd and Laframboise, Math. Comp. 36, 1981; K = 4, degree 13, Chebyshev points for x up to
// 4: 4e-16 of the value; less beyond that, of a value below 1e-8).  Root mean square error against 60 digits, and of the library's erf
// in td_act_f64: 6.5e-17 and 7.5e-17 for z from N(0, 1.6^2), 2.66e-17 and 2.72e-17 from N(0, 0.6^2), 1.7e-16 and 2.0e-16 for z from -8 to 8.
// a b + c with the constant c in scalar registers.  (Left to the compiler a step of a polynomial is two moves of c into the registers
// that v_fmac_f64 then adds to: 126 instead of 75 vector instructions
// for a sample's sigma and sums in the calibration's fit.)
__device__ __forceinline__ double fma_constant(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}
__device__ __forceinline__ double rcp_f64(double a) {              // a: a normal number
    double r = __builtin_amdgcn_rcp(a);
    r = fma(fma(-a, r, 1.0), r, r);
    return fma(fma(-a, r, 1.0), r, r);
}
// N values side by side, so that N steps of a polynomial share their constant
template <int N> __device__ __forceinline__ void step_f64(double (&s)[N], const double (&x)[N], double c) {
#pragma unroll
    for (int u = 0; u < N; ++u) s[u] = fma_constant(s[u], x[u], c);
}
template <int N> __device__ __forceinline__ void exp_f64(double (&y)[N]) {   // |y| <= 2^20: Taylor's series, 13 terms, on |r| <= log(2) / 2
    // log(2): its first 30 bits, so that n times them is exact; the rest
    constexpr double kHead = 0.6931471796706319, kRest = 8.893134238886677e-10;
    constexpr double c[13] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
                              1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600};
    double n[N], s[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        n[u] = rint(y[u] * 1.4426950408889634074);
        y[u] = fma(n[u], -kRest, fma(n[u], -kHead, y[u]));
        s[u] = c[12];
    }
#pragma unroll
    for (int k = 11; k >= 3; --k) step_f64(s, y, c[k]);
#pragma unroll
    for (int u = 0; u < N; ++u) y[u] = ldexp(fma(fma(fma(s[u], y[u], 0.5), y[u], 1.0), y[u], 1.0), (int)n[u]);   // (these constants the instruction has)
}
template <int ACT, int N> __device__ __forceinline__ void act_flat_f64(double (&z)[N]) {
    if constexpr (ACT == TARDIS_ACT_GELU_ERF) {
        constexpr double K = 4.0, kRootHalf = 0.70710678118654752440;
        constexpr double c[14] = {                                         // (of half the function)
            0.4692779762826495, -0.2957906600056251, 0.16285305891539317, -0.07694746904507938, 0.03026111138288409,
            -0.009324134291590786, 0.0019168261198674933, -8.089792150921698e-05, -0.00011294695657629944,
            2.652979050688696e-05, -6.266870568616483e-06, -8.396392546762074e-06, -1.6994783085984142e-06,
            -8.019930824959331e-08};
        constexpr double b[10] = {
            0.39894228040143265, -0.06649038006690387, 0.009973557009983732, -0.001187328214811527, 0.0001154346832492605,
            -9.444639861853272e-06, 6.659317805752481e-07, -4.117317843452298e-08, 2.2271240384729976e-09,
            -9.027164883791298e-11};
        double u[N], w[N], near[N], half[N];
        bool far = false;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            u[i] = fmin(fabs(z[i]), 60.0);                                 // (Phi(-60) is 0, and infinities stay what they were)
            w[i] = u[i] * u[i];
            near[i] = b[9];
            half[i] = 0.0;
            far |= u[i] >= 1.0;
        }
#pragma unroll
        for (int k = 8; k >= 0; --k) step_f64(near, w, b[k]);
        if (__any(far)) {                                                  // (a layer's samples may all lie below 1)
            double r[N], t[N], s[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                r[i] = rcp_f64(fma_constant(u[i], kRootHalf, K - kRootHalf));
                t[i] = fma(-2.0 * K, r[i], 1.0);
                s[i] = c[13];
                w[i] *= -0.5;
            }
#pragma unroll
            for (int k = 12; k >= 0; --k) step_f64(s, t, c[k]);
            exp_f64(w);
#pragma unroll
            for (int i = 0; i < N; ++i) half[i] = s[i] * r[i] * w[i];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) z[i] *= u[i] < 1.0 ? fma(z[i], near[i], 0.5) : z[i] > 0.0 ? 1.0 - half[i] : half[i];
    } else if constexpr (ACT == TARDIS_ACT_GELU_TANH) {
        // as in 32 bits; |v| beyond 1e5 is 1e5 (where e is 0)
        double e[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double v = 0.79788456080286535588 * (z[i] + 0.044715 * z[i] * z[i] * z[i]);
            e[i] = fmax(-2.0 * fabs(v), -1e5);
        }
        exp_f64(e);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double q = e[i] * rcp_f64(1.0 + e[i]);
            z[i] *= z[i] > 0.0 ? 1.0 - q : q;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) z[i] = td_act_f64(z[i], ACT);
    }
}
template <int ACT> __device__ __forceinline__ double act_flat_f64(double z) {
    double v[1] = {z};
    act_flat_f64<ACT>(v);
    return v[0];
}
