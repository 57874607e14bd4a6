// The gate functions of the LSTM cells in the resident decode kernel.
#pragma once
#include <hip/hip_runtime.h>

namespace rnnt {

// sigmoid(x), or tanh(x) where th, as base - N / D.  With e = exp(-|x|) or exp(-2 |x|), D = 1 + e:
// tanh is +-(1 - 2 e / D), the sigmoid 1 - e / D or, below zero, -(-e / D), so the quotient's error counts
// in full only where it is the whole result.  tanh below 0.7 is Lambert's continued fraction to x^5 / x^4,
// written as x less a correction of at most a sixth of it (1 - 2 e / D would cancel there; the fraction
// is cut off 0.04 units in the last place from tanh at 0.7).
// The exponential is the hardware's exp2, 2^t, corrected by what the rounding of t leaves; the quotient is the
// hardware's reciprocal and a residual, v + f v - n with D = 1 + f, that is free of the rounding of D.  (Fused by
// the compiler, n - v would be n - n r: no contractions here but those written.)
// Over all floats, against 64 bits: at most 2.58 units in the last place for the sigmoid (down to -87; below
// it stays at 1.6e-38) and 1.21 for tanh, where 1 / (1 + expf(-x)) and tanhf have 2.63 and 1.41.  The quotient
// as the whole result, without the residual's care: 3.47 and 2.87 at 33 vector instructions instead of 34;
// the exponential's correction carried into the residual: 1.75 and 1.04 at 40, 0.05 us a cell.
// NaN stays NaN: the limit is the minimum that passes it on.
__device__ __forceinline__ float gate_act(float x, bool th)
{
#pragma clang fp contract(off)
    const float m = th ? 2.f : 1.f;
    const float y = __builtin_elementwise_minimum(fabsf(x * m), 87.f);
    const float t = -y * 1.44269504f;                                                     // log2(e)
    float e = __builtin_amdgcn_exp2f(t);
    e = fmaf(e, fmaf(-t, -1.90465421e-9f, fmaf(-t, 0.693147182f, -y)), e);                // -t ln(2) - y
    const float q = x * x, sm = copysignf(m, x);
    const bool small = th && fabsf(x) < 0.7f;
    float n = e * sm, f = e, base = fmaf(sm, 0.5f, th ? 0.f : 0.5f);
    n = small ? x * q * fmaf(q, 14.f, 315.f) : n;
    f = small ? fmaf(q, fmaf(q, 15.f, 420.f), 944.f) : f;
    base = small ? x : base;
    const float r = __builtin_amdgcn_rcpf(1.f + f), v = n * r;
    return base - fmaf(fmaf(-f, v, n - v), r, v);
}

}  // namespace rnnt
