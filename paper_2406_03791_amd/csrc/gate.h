// The gate functions of the LSTM cells in the resident decode kernel.
#pragma once
#include <hip/hip_runtime.h>

namespace rnnt {

// sigmoid(x), or tanh(x) where th: both are N / (1 + e) with e = exp(-x) or exp(-2x); tanh below
// 0.55, where 1 - e would cancel, is Lambert's continued fraction to x^5 / x^4.  The exponential is
// the hardware's exp2 with the rounding of x log2(e) carried along, the quotient the hardware's
// reciprocal with two Newton steps; at most 3 units in the last place over the whole range.  NaN stays
// NaN: the limits are the minimum and maximum that pass it on.
__device__ __forceinline__ float gate_act(float x, bool th)
{
    const float y = __builtin_elementwise_minimum(__builtin_elementwise_maximum(th ? x + x : x, -80.f), 80.f);
    const float kL = 1.44269504f, kLo = 1.92596303e-8f;          // log2(e)
    const float t = -y * kL;
    const float lo = fmaf(-y, kL, -t) - y * kLo;
    float e = __builtin_amdgcn_exp2f(t);
    e = fmaf(e, lo * 0.693147182f, e);
    const float q = x * x;
    const bool small = th && fabsf(x) < 0.55f;
    float n = th ? 1.f - e : 1.f, d = 1.f + e;
    n = small ? x * fmaf(q, 105.f + q, 945.f) : n;
    d = small ? fmaf(q, fmaf(q, 15.f, 420.f), 945.f) : d;
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(fmaf(-d, r, 1.f), r, r);
    const float v = n * r;
    return fmaf(fmaf(-d, v, n), r, v);
}

}  // namespace rnnt
