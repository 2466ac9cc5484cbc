// Device helpers shared by the prompt-sized kernels (prefill_kernels.hip, prefill_gemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "device_utils.h"
#include "prefill_params.h"

namespace cfpp {

__device__ __forceinline__ void pf_split(float v, __half &hi, __half &lo)
{
    hi = __float2half_rn(v);
    lo = __float2half_rn(v - __half2float(hi));
}

__device__ __forceinline__ unsigned pf_pack2(float a, float b)
{
    return (unsigned)__half_as_ushort(__float2half_rn(a)) | (unsigned)__half_as_ushort(__float2half_rn(b)) << 16;
}

// GELU for the GEMM epilogues, where its instructions are what a tile waits for (the library's erff
// takes about three times as many): with x = |z| and t = 1 / (1 + x / 2),
//   Phi(-x) = erfc(x / sqrt 2) / 2 = t P(t) exp(-x^2 / 2),   gelu(z) = z (z < 0 ? Phi(-x) : 1 - Phi(-x)),
// P a degree-7 fit (weighted least squares on Chebyshev nodes, reweighted towards the minimax) of
// erfcx(x / sqrt 2) / (2 t).  Against 64 bits, z in [-9, 9]: largest error 3.84e-7, relative 2-norm over
// N(0, 1) 3.6e-8, where z (1 + erf) / 2 in 32 bits with a correctly rounded erf has 4.47e-7 and 3.7e-8
// (and loses the negative tail to cancellation).  The tanh form as z / (1 + exp(-2 u)).
__device__ __forceinline__ float pf_gelu(float z, int flags)
{
    if (flags & kFlagTanhGelu) {
        const float u = 0.79788456080286535588f * (z + 0.044715f * z * z * z);
        return z * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-2.8853900817779268f * u));
    }
    const float x = fabsf(z), t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.f));
    float p = 0.0235918909f;
    p = fmaf(p, t, -0.168402344f);
    p = fmaf(p, t, 0.490389824f);
    p = fmaf(p, t, -0.700354338f);
    p = fmaf(p, t, 0.396986157f);
    p = fmaf(p, t, 0.0420736447f);
    p = fmaf(p, t, 0.217516899f);
    p = fmaf(p, t, 0.198198274f);
    const float q = t * p * __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);
    return z * (z < 0.f ? q : 1.f - q);
}

// Where the head of element k of a row lies in an activation buffer of `width` values a row
// (interleaved planes, prefill_params.h); its remainder is kPfLo halves further.
constexpr int kPfLo = 32;
__device__ __forceinline__ size_t pf_at(int row, int k, int width)
{
    return (size_t)row * pf_row_halves(width) + (k >> 5) * 64 + (k & 31);
}

}  // namespace cfpp
