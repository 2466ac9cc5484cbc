// The attention of a short prompt with MLP-down in the same launch (prefill_attention.h): its instances by head size and sets of tokens.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "prefill_attention.h"

namespace cfpp {

template <int D, bool SPLIT, int S>
static hipError_t beside(const PfParams &P, const PfAttnParts &A, hipStream_t s)
{
    constexpr int QW = D == 128 ? 2 : 1, lds = pf_attn_lds<D, QW>() > pf_down_lds<S>() ? pf_attn_lds<D, QW>() : pf_down_lds<S>();
    const hipError_t e = hipFuncSetAttribute((const void *)k_pf_attn<D, QW, SPLIT, S>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    const int groups = (P.dm.h + 16 * pf_down_tiles<S>() - 1) / (16 * pf_down_tiles<S>());
    hipLaunchKernelGGL((k_pf_attn<D, QW, SPLIT, S>), dim3(A.first_down + groups * P.nrw.downs), dim3(256), lds, s, P, A);
    return hipGetLastError();
}
template <int D, bool SPLIT>
static hipError_t sets(const PfParams &P, const PfAttnParts &A, hipStream_t s)
{
    switch ((P.n_rows + 7) / 8) {
    case 1: return beside<D, SPLIT, 1>(P, A, s);
    case 2: return beside<D, SPLIT, 2>(P, A, s);
    case 3: return beside<D, SPLIT, 3>(P, A, s);
    case 4: return beside<D, SPLIT, 4>(P, A, s);
    case 5: return beside<D, SPLIT, 5>(P, A, s);
    case 6: return beside<D, SPLIT, 6>(P, A, s);
    }
    return hipErrorInvalidValue;
}
template <int D>
static hipError_t split(const PfParams &P, const PfAttnParts &A, hipStream_t s) { return A.parts > 1 ? sets<D, true>(P, A, s) : sets<D, false>(P, A, s); }

hipError_t launch_pf_attention_beside(const PfParams &P, const PfAttnParts &A, hipStream_t s)
{
    switch (P.dm.d) {
    case 64: return split<64>(P, A, s);
    case 80: return split<80>(P, A, s);
    case 128: return split<128>(P, A, s);
    }
    return hipErrorInvalidValue;
}

int pf_down_rows(int tokens) { return 16 * ((tokens + 7) / 8 <= 5 ? pf_down_tiles<5>() : pf_down_tiles<6>()); }

// Parts of K: 640 columns to one or more, and one workgroup to a CU, or two where that is more than 256 KiB of weights to one (hidden 1280, 21 tokens
// in five / eight parts: 25.5 / 24.5 us a layer; 2560, 8 tokens in six / twelve 39.4 / 39.9).  Not taken, 0, where the sets' activations are too much
// beside the weights: every workgroup reads those of its part from the L2, and a ring that holds them holds fewer weights.  us a layer, both
// products behind the attention -> this: hidden 512, 8 / 30 tokens 17.1 -> 15.9 / 19.1 -> 18.8; 1024, 13 / 37 / 44 22.1 -> 20.1 / 26.7 -> 24.2 / 27.9 -> 25.2;
// 1280, 8 / 37 23.3 -> 21.1 / 30.0 -> 28.3; 1536, 8 / 30 25.1 -> 23.8 / 30.7 -> 29.9, but 44 34.2 -> 34.3; 2560, 8 / 13 / 21 41.3 -> 39.4 / 43.7 -> 42.8 / 46.5
// -> 46.5, but 37 / 44 53.9 -> 54.2 / 59.3 -> 63.1; 4096, 8 / 13 81.3 -> 76.2 / 83.8 -> 81.8, but 30 97.5 -> 99.1.  Five sets of small hidden sizes are
// 12 or 24 workgroups of 64 rows: 36 tokens from an empty cache / behind 1000 / 2000 positions, hidden 384 18.7 -> 19.5 / 24.5 -> 23.8 / 24.0 -> 24.1, 512 19.7 -> 20.0 /
// 25.4 -> 24.0 / 24.6 -> 24.1; from 640 on they gain: 640 (80) 22.9 -> 21.6 / 30.8 -> 29.3 / 30.2 -> 28.7, 640 (64) 22.0 -> 21.5 / 27.9 -> 26.1 / 27.7 -> 26.9, 768
// 22.9 -> 22.5 / 28.9 -> 26.8 / 28.6 -> 27.6, 1024 (128) 26.8 -> 24.2 / 35.1 -> 32.1 / 36.1 -> 33.4, 1280 (80) 30.0 -> 28.3 / 38.0 -> 37.6 / 37.7 -> 38.5, 1536
// 32.3 -> 31.7 / 38.3 -> 38.2 / 40.1 -> 38.9, but 1024 (64) 24.9 -> 24.1 / 30.7 -> 28.2 / 30.6 -> 31.1.  (Where the context lies does not enter: the same
// tokens are added in the same order wherever they stand.)
int pf_down_parts(const Dims &dm, int tokens)
{
    const int sets = (tokens + 7) / 8;
    if (sets > 6 || (sets > 2 && sets * dm.h > 7680)) return 0;
    if (sets == 5 && dm.h < 640) return 0;
    const int rows = pf_down_rows(tokens), per_cu = (size_t)dm.h * dm.f * 2 > (size_t)256 * 256 * 1024 ? 2 : 1;
    return min(min(kPfDownParts, max(1, dm.f / 640)), max(1, per_cu * 256 * rows / dm.h));
}

}  // namespace cfpp
