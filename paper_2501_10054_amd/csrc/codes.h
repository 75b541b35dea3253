// Predictor codes of 8 bits from bf16 weights in 32-bit arithmetic: code = rint(w * scale), as one fma onto 1.5 * 2^23, whose low byte it
// is.  For host and device, so that it can be compared with the definition on a CPU.
#pragma once
#include <cmath>
#include <cstdint>

#include "slices.h"

// The scale with which the codes of a row of bf16 numbers, whose largest magnitude is m, are those of the definition,
// rint(w / s) with s = m / 127 in 64 bits.  half: the code that the definition gives m / 2.
// With weights of 8 significant bits, w = a 2^x and m = b 2^y, the quotient 127 a 2^(x-y) / b is a half of an odd number or by 1 / (254 a) > 1.5e-5
// of itself away from one, which two units in the last place of the scale do not bridge.  It is a half itself where
// b = 254 - then s is a power of two, the scale is exact and so is either form's tie - and for a = b 2^n with a quotient of 127 / 2^n, which
// is one for n = 1: w = m / 2.  What the definition makes of that depends on how s was rounded; the scale is chosen to its side.
TD_HD float td_code_scale(float m, int half) {
    float scale = (float)(127.0 / (double)m);
    const float up = half == 64 ? INFINITY : 0.0f;
    while ((0.5 * (double)m * (double)scale >= 63.5) != (half == 64)) scale = nextafterf(scale, up);
    return scale;
}

TD_HD uint32_t td_code_bits(float w, float scale) {                // low byte: the code
    union { float f; uint32_t u; } v;
    v.f = fmaf(w, scale, 12582912.0f);
    return v.u;
}
