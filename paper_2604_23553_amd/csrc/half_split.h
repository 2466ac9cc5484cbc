// An fp32 value as two fp16 values, head and remainder: what the matrix-core paths feed the fp16 instruction in turn.
// v = hi + lo to 2^-22 |v| or, where the remainder is subnormal, to 2^-25; from 65520 on the head is infinite and the two are NaN
// together.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

namespace cfpp {

// Head and remainder have to come from one rounding.  Where v is a product the compiler may round it to fp16 at once in
// one place (v_fma_mixlo) and to fp32 and then to fp16 in another; for one value in some thousands the two heads differ
// by a step, and a remainder formed from one does not belong to the other: the value is then off by 2^-11.  So the value
// is one register, whatever it was computed from.
__device__ __forceinline__ float split_value(float v)
{
    asm("" : "+v"(v));
    return v;
}
__device__ __forceinline__ void split_half(float value, __half &hi, __half &lo)
{
    const float v = split_value(value);
    hi = __float2half_rn(v);
    lo = __float2half_rn(v - __half2float(hi));
}

}  // namespace cfpp
