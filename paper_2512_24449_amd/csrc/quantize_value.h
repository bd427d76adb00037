// Token-wise quantization of one value (PackKV Sec. III-B.2), for kernels and for checks on the host.
#pragma once

#include <math.h>

namespace packkv {

// The code of a value with the token's scale and minimum:
// clamp(rint(fl((x - mn) / s)), 0, qmax), the quotient rounded to fp32 as an IEEE divide does.
// r is the token's 1 / s from an IEEE divide (once per token).  The product (x - mn) * r lies
// within 1.5 * 2^-23 relative of that rounded quotient (half an ulp for r, half for the product,
// half for the quotient's own rounding), which is below 5e-5 in absolute terms for every quotient
// that is not clamped anyway (<= 256.5; beyond that both round to at least 256 > qmax).  So unless
// the product is within 1e-3 of a rounding tie k + 0.5, rint of the product IS rint of the
// quotient; the rare value near a tie takes the divide.
// A quotient that is no number (NaN or infinite values) takes qmax, as in the other rules (quantize_token8, quantize_quad in
// compress.hip): a chunk sized by one of them and written by another must come out the same.
__host__ __device__ inline int quantize_value(float x, float s, float mn, float r, int qmax) {
    int v = 0;
    if (s != 0.0f) {
        const float a = x - mn;
        const float q1 = a * r;
        float t = rintf(q1);  // ties to even
        if (fabsf(fabsf(q1 - t) - 0.5f) < 1e-3f) t = rintf(a / s);  // IEEE fp32 divide
        v = (int)fmaxf(fminf(t, float(qmax)), 0.0f);
    }
    return v;
}

}  // namespace packkv
