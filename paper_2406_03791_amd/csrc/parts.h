// fp32 values as two fp16 parts each, for the 16-bit matrix instructions (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace rnnt {

// Two fp32 values as fp16 parts (ties to even), the first in the low half: the nearest fp16 numbers, and those nearest
// to what is left.  (v_fma_mixlo_f16 and v_fma_mixhi_f16 would do each of the four in one instruction, but they write
// half a register and take twice the time of others: 8.7 cycles against 4.3 to 4.9.)
__device__ __forceinline__ unsigned f16_pair(float a, float b)
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, h2));
}
__device__ __forceinline__ void f16_parts(float a, float b, unsigned &high, unsigned &low)
{
    high = f16_pair(a, b);
    // (in instructions that take the fp16 number as it is: from C++ a conversion and a subtraction come)
    float ra, rb;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(ra) : "v"(a), "v"(high));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(rb) : "v"(b), "v"(high));
    low = f16_pair(ra, rb);
}
// two fp32 values as bf16 (ties to even), first in the low half
__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, b2));
}

}  // namespace rnnt
