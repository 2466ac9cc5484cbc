// Device helpers shared by the prompt-sized kernels (prefill_kernels.hip, prefill_gemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "device_utils.h"
#include "half_split.h"
#include "prefill_params.h"
#include "narrow_params.h"

namespace cfpp {

__device__ __forceinline__ unsigned pf_pack2(float a, float b)
{
    return (unsigned)__half_as_ushort(__float2half_rn(a)) | (unsigned)__half_as_ushort(__float2half_rn(b)) << 16;
}

// GELU for the GEMM epilogues, where its instructions are what a tile waits for (with the library's erff and tanhf:
// 512 tokens at hidden 2560 + 2 %, 1531 at hidden 4096 with the tanh form + 4 % of the whole pass).
// gelu(z) = z Phi(z), with x = |z|, y = z^2:
//   x < 0.85:  Phi(z) = 1/2 + z R(y), R of degree 4;
//   else:   Phi(-x) = q, Phi(x) = 1 - q;  erf form: q = erfc(x / sqrt 2) / 2 = t P(t) exp(-y / 2), t = 1 / (1 + x / 2), P of
//           degree 7;  tanh form: q = e / (1 + e), e = exp(-2 u), u = sqrt(2 / pi) (x + 0.044715 x^3).
// P fits erfcx(x / sqrt 2) / (2 t), R (Phi(z) - 1/2) / z (weighted least squares on Chebyshev nodes, reweighted towards the
// minimax).  Near zero q alone is not good enough: Phi(z) = 1 - q carries the rounding of q's factors, which 1 + erf does not.
// Measured against 64 bits, largest error and relative 2-norm, the library's forms -> these:
//   erf:  N(0, 0.3) 1.17e-7, 4.09e-8 -> 0.92e-7, 3.71e-8;  N(0, 1) 4.16e-7, 3.85e-8 -> 3.43e-7, 3.36e-8;  [-9, 9] 4.47e-7, 1.75e-8 -> 3.84e-7, 1.56e-8
//   tanh: N(0, 0.3) 1.11e-7, 4.10e-8 -> 0.93e-7, 3.71e-8;  N(0, 1) 3.57e-7, 3.76e-8 -> 3.50e-7, 3.35e-8;  [-9, 9] 4.33e-7, 1.57e-8 -> 3.65e-7, 1.41e-8
__device__ __forceinline__ float pf_gelu(float z, int flags)
{
    const float x = fabsf(z), y = z * z;
    float q, r;
    if (flags & kFlagTanhGelu) {
        const float e = __builtin_amdgcn_exp2f(-x * fmaf(0.10294324f, y, 2.3022082f));
        q = e * __builtin_amdgcn_rcpf(1.f + e);
        r = fmaf(1.03582883e-4f, y, -0.00123273977f);
        r = fmaf(r, y, 0.0101983044f);
        r = fmaf(r, y, -0.0668190569f);
        r = fmaf(r, y, 0.398942262f);
    } else {
        const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.f));
        float p = 0.0235918909f;
        p = fmaf(p, t, -0.168402344f);
        p = fmaf(p, t, 0.490389824f);
        p = fmaf(p, t, -0.700354338f);
        p = fmaf(p, t, 0.396986157f);
        p = fmaf(p, t, 0.0420736447f);
        p = fmaf(p, t, 0.217516899f);
        p = fmaf(p, t, 0.198198274f);
        q = t * p * __builtin_amdgcn_exp2f(y * -0.72134752044448170f);
        r = fmaf(9.82774509e-5f, y, -0.00117531931f);
        r = fmaf(r, y, 0.00996982493f);
        r = fmaf(r, y, -0.0664899051f);
        r = fmaf(r, y, 0.398942262f);
    }
    return z * (x < 0.85f ? fmaf(z, r, 0.5f) : z < 0.f ? q : 1.f - q);
}

// Where the head of element k of a row lies in an activation buffer of `width` values a row
// (interleaved planes, prefill_params.h); its remainder is kPfLo halves further.
constexpr int kPfLo = 32;
__device__ __forceinline__ size_t pf_at(int row, int k, int width)
{
    return (size_t)row * pf_row_halves(width) + (k >> 5) * 64 + (k & 31);
}
// The same in the order that the pass's products read, and the distance of the remainder.
__device__ __forceinline__ size_t pf_out_at(const PfParams &P, int row, int k, int width)
{
    return P.nrw.on ? ng_at(row, k, width, kNgSet) : pf_at(row, k, width);
}
__device__ __forceinline__ int pf_out_lo(const PfParams &P) { return P.nrw.on ? 8 * kNgSet : kPfLo; }

}  // namespace cfpp
