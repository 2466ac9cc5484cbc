// Prompt processing with the weights read once per pass over up to kPfMaxRows
// tokens (the paper names a prefill phase beside its fused decode kernel, Sec. 4.2;
// what is computed is the block of Sec. 2.2 applied to every prompt token with
// causal attention).  With hundreds of tokens the projections are dense
// contractions - tokens x K activations times K x rows weights - and run as
// LDS-tiled GEMMs on the matrix cores (prefill_gemm.hip); the attention of
// a pass reads the cache rows its own QKV launch appended.
//
//   k_pf_row<>  : per token: (the previous layer's output from the parts of its product,)
//                 mean, 1/sigma, and gamma_1 * x, gamma_2 * x as two fp16 planes each (head +
//                 remainder: y = hi + lo (half_split.h), so that the fp16 matrix instruction
//                 reproduces the fp32 product to rounding)
//   the products: prefill_gemm.hip - QKV and MLP-up in one launch, output projection and
//                 MLP-down as one product
//   k_pf_attn<> : (prefill_attention.h) causal attention of a block of 32, 64 or 128 queries of one head over the
//                 cache, keys in LDS tiles, both products on the matrix cores
//                 (v_mfma_f32_32x32x16_f16), online softmax in fp32; of a short prompt with MLP-down in the same
//                 launch (prefill_beside.hip)
//
// Every sum has a fixed order: one bit pattern per build and pass size.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "prefill_attention.h"

namespace cfpp {

// ---------------------------------------------------------------------------
// What a layer's first product reads, for one token: the layer input x, its mean and 1/sigma, and
// gamma_1 * x, gamma_2 * x as head and remainder planes.  256 threads a token, a thread holds the
// elements 4 (tid + 256 j) .. + 3, j < h / 1024 (hidden: a multiple of 128, at most 4096).  Rows
// past the pass's tokens are left alone: what a product makes of them is never stored.
// FROM_PARTS: x is the previous layer's output, still in the parts of its second product - the parts
// are added in order, biases and residual follow, and the row goes to the residual stream (and, as
// the last layer's output, to out) on the way: one launch where the sum and the LayerNorm were two
// (512 tokens of the 2560-wide shape: 10.1 + 10.2 us).  Bound by the latency of a row's loads and
// stores, hence four or sixteen wavefronts to a row.
// With few tokens there is one row to a CU and what counts is how many trips to memory follow one another: 1024 threads
// to a row, one float4 each, all its parts in flight together (37 tokens of hidden 2560, 8 parts: 7.8 us with 256
// threads, 5.6; 128 tokens, whole layer: 106.1, 104.0).  Up to kPfRowWide tokens; from about 1000 on 256 threads are faster (hidden
// 512, 1000 tokens, layer: 51.3 against 53.0), in between the two are within 1 % of a layer.
constexpr int kPfRowVec = 4;           // float4 per thread of 256: hidden <= 4096
constexpr int kPfRowWide = 256;
template <bool FROM_PARTS, int NT>
__global__ void __launch_bounds__(NT) k_pf_row(PfParams P)
{
    constexpr int VEC = 1024 / NT, NW = NT / 64;
    __shared__ float red[2][NW];
    const Dims &dm = P.dm;
    const int h = dm.h, nv = h >> 2, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = blockIdx.x;
    const bool last = FROM_PARTS && P.layer == P.n_layers - 1, bare = last || (FROM_PARTS && !P.row_fused);   // bare: no LayerNorm here
    const __half *wn = FROM_PARTS ? P.w_next : P.w;        // the layer whose LayerNorms these are
    f32x4 x[VEC];
    uint2 g1[VEC], g2[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const int g = tid + NT * j;
        x[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (g >= nv) continue;
        const size_t at = (size_t)row * h + 4 * g;
        if (!bare) {
            g1[j] = *reinterpret_cast<const uint2 *>(wn + P.lay.ln1_g + 4 * g);
            g2[j] = *reinterpret_cast<const uint2 *>(wn + P.lay.ln2_g + 4 * g);
        }
        if (FROM_PARTS) {
            const size_t zstride = P.part_out_stride;
            const float *p = P.part_out + at;
            const f32x4 r = *as_global(reinterpret_cast<const f32x4 *>(P.xres + at));
            const uint2 de = *reinterpret_cast<const uint2 *>(P.w + P.lay.b_dense + 4 * g), dn = *reinterpret_cast<const uint2 *>(P.w + P.lay.b_down + 4 * g);
            f32x4 s = *as_global(reinterpret_cast<const f32x4 *>(p));
            const int splits = P.plan_out.splits;
            constexpr int AT = NT == 1024 ? 9 : 5;         // parts requested at a time (past the last: the last again)
            for (int z = 1; z < splits; z += AT) {
                f32x4 t[AT];
#pragma unroll
                for (int u = 0; u < AT; ++u) t[u] = *as_global(reinterpret_cast<const f32x4 *>(p + min(z + u, splits - 1) * zstride));
#pragma unroll
                for (int u = 0; u < AT; ++u)
                    if (z + u < splits) s += t[u];
            }
            const float2 de0 = unpack_h2(de.x), de1 = unpack_h2(de.y), dn0 = unpack_h2(dn.x), dn1 = unpack_h2(dn.y);
            x[j][0] = r[0] + ((s[0] + de0.x) + dn0.x);
            x[j][1] = r[1] + ((s[1] + de0.y) + dn0.y);
            x[j][2] = r[2] + ((s[2] + de1.x) + dn1.x);
            x[j][3] = r[3] + ((s[3] + de1.y) + dn1.y);
            if (last) {
                uint2 o;
                o.x = pf_pack2(x[j][0], x[j][1]); o.y = pf_pack2(x[j][2], x[j][3]);
                *reinterpret_cast<uint2 *>(P.out + at) = o;
            } else {
                *reinterpret_cast<f32x4 *>(P.xnext + at) = x[j];
            }
        } else if (P.layer == 0) {
            const uint2 w = *reinterpret_cast<const uint2 *>(P.x_in + at);
            const float2 a = unpack_h2(w.x), b = unpack_h2(w.y);
            x[j] = f32x4{a.x, a.y, b.x, b.y};
            *reinterpret_cast<f32x4 *>(P.xres + at) = x[j];
        } else {
            x[j] = *reinterpret_cast<const f32x4 *>(P.xres + at);
        }
    }
    if (bare) return;                                      // (uniform)
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) s += (x[j][0] + x[j][1]) + (x[j][2] + x[j][3]);
    s = wave_sum(s);
    if (lane == 0) red[0][wave] = s;
    __syncthreads();
    float total = red[0][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) total += red[0][w];
    const float mean = total / (float)h;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        if (tid + NT * j < nv) {
            const f32x4 dl = x[j] - mean;
            q += (dl[0] * dl[0] + dl[1] * dl[1]) + (dl[2] * dl[2] + dl[3] * dl[3]);
        }
    }
    q = wave_sum(q);
    if (lane == 0) red[1][wave] = q;
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const int g = tid + NT * j;
        if (g >= nv) continue;
        const float2 a1 = unpack_h2(g1[j].x), b1 = unpack_h2(g1[j].y), a2 = unpack_h2(g2[j].x), b2 = unpack_h2(g2[j].y);
        const float ga[4] = {a1.x, a1.y, b1.x, b1.y}, gb[4] = {a2.x, a2.y, b2.x, b2.y};
        __half h1[4], l1[4], h2[4], l2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            split_half(x[j][e] * ga[e], h1[e], l1[e]);
            split_half(x[j][e] * gb[e], h2[e], l2[e]);
        }
        const size_t at = pf_out_at(P, row, 4 * g, h), al = at + pf_out_lo(P);
        *reinterpret_cast<uint2 *>(P.y1 + at) = *reinterpret_cast<const uint2 *>(h1);
        *reinterpret_cast<uint2 *>(P.y1 + al) = *reinterpret_cast<const uint2 *>(l1);
        *reinterpret_cast<uint2 *>(P.y2 + at) = *reinterpret_cast<const uint2 *>(h2);
        *reinterpret_cast<uint2 *>(P.y2 + al) = *reinterpret_cast<const uint2 *>(l2);
    }
    __syncthreads();
    if (tid == 0) {
        float sq = red[1][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) sq += red[1][w];
        P.stats[row] = float2{mean, 1.0f / sqrtf(sq / (float)h + dm.ln_eps)};
    }
}

// The parts of a split attention, added in order: a workgroup per head and block of 32 queries.  (A query's output may carry
// a later token's V from up to 127 positions behind the block's first: those that k_pf_attn's largest block holds.)
template <int D>
__global__ void __launch_bounds__(256) k_pf_attn_join(PfParams P, PfAttnParts A)
{
    const Dims &dm = P.dm;
    const int head = blockIdx.x, q0 = (int)blockIdx.y * 32;
    const __half *Kc = P.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vc = P.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    pf_attn_finish<D, 1>(P, Kc, Vc, head, q0, P.pos0 + min(q0 + 128, P.n_rows) - 1, threadIdx.x, [&](int q, int c8, f32x4 (&v)[2]) {
        constexpr int AT = 8;                              // parts requested at a time (past the last: the last again)
        float m = -INFINITY, l = 0.f;
        v[0] = v[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int z = 0; z < A.parts; z += AT) {
            float2 ml[AT];
            f32x4 a[AT], b[AT];
#pragma unroll
            for (int u = 0; u < AT; ++u) {
                const size_t row = (size_t)min(z + u, A.parts - 1) * P.n_rows + q0 + q;
                ml[u] = A.ml[row * dm.H + head];
                const f32x4 *o = reinterpret_cast<const f32x4 *>(A.o + row * dm.h + head * D + c8);
                a[u] = o[0]; b[u] = o[1];
            }
            float mn = m;
#pragma unroll
            for (int u = 0; u < AT; ++u) mn = fmaxf(mn, ml[u].x);
            const float c0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
            l *= c0; v[0] *= c0; v[1] *= c0;
#pragma unroll
            for (int u = 0; u < AT; ++u) {
                if (z + u >= A.parts) continue;            // (uniform)
                const float c = ml[u].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - mn);
                l = fmaf(ml[u].y, c, l);
                v[0] += a[u] * c; v[1] += b[u] * c;
            }
            m = mn;
        }
        return l;
    });
}

// ---------------------------------------------------------------------------
bool pf_supported(const Dims &dm)
{
    return dm.h % kPfTile == 0 && dm.f % kPfTile == 0 && dm.h <= 1024 * kPfRowVec && (dm.d == 64 || dm.d == 80 || dm.d == 128) &&
           !(dm.flags & kFlagSequentialResidual) && dm.r % 2 == 0;
}

// Queries per workgroup: a tile of K and V is fetched and transposed once per workgroup, so as many as leave the
// chip filled; with fewer, the wavefronts split the keys instead.  By n = heads x blocks of 32 queries, us per layer
// with 1 / 2 / 4 blocks of 32 (LayerNorm and products included): D = 80: n = 512 (3000 positions cached) 258 / 262 / 287,
// 768: 288 / 287 / 291, 1024: 380 / 376 / 382, 2048: 689 / 681 / 678; D = 64: n = 128: 46 / 50 / 53, 1024: 145 / 148 / 172;
// D = 128: n = 64 (3000 cached) 222 / 202 / 228, 1024: 785 / 762 / 768, 1536: 4 blocks 6 us faster than 2 (one block's
// tile of 128 keys spills registers there and is not built).
// Kernel times before (16 queries to a workgroup, 64 from 1024 tokens, 16x16x16 instructions) -> now: hidden 2560, 512
// tokens 23 -> 16 us, 4096 tokens 370 -> 227; hidden 4096, 1531 tokens behind 700: 221 -> 126.
// Parts of the keys: as many as leave every CU a workgroup and each part two tiles, if a workgroup saves at least five
// tiles (1.3 us each) by it: the launch that adds the parts takes 4 - 5 us.  us per layer, whole -> in parts: hidden 2560: 1
// token behind 1000 / 3000 51.6 -> 48.1 / 73.3 -> 49.9, 37 tokens 65.7 -> 63.4 / 86.4 -> 67.5, 128 tokens behind 3000 143 -> 131;
// hidden 4096, 37 tokens 120 -> 109 / 160 -> 114; hidden 512, 37 tokens 29.4 -> 28.0 / 44.8 -> 26.7.  With more (16 parts, or
// two workgroups to a CU) the parts' traffic and the join cost what the shorter walks save.
constexpr int kPfAttnPartsMax = 8;
static int pf_attn_blocks(const Dims &dm, int tokens)                  // blocks of 32 queries to a workgroup
{
    const int n = dm.H * ((tokens + 31) / 32);
    return n >= (dm.d == 128 ? 1536 : 2048) ? 4 : dm.d == 128 || n >= 768 ? 2 : 1;
}
int pf_attn_parts(const PfParams &P)
{
    const int qw = pf_attn_blocks(P.dm, P.n_rows);
    if (qw != (P.dm.d == 128 ? 2 : 1)) return 1;           // (with more queries to a workgroup there are more workgroups than CUs)
    const int tk = 128 / qw, wgs = P.dm.H * ((P.n_rows + 32 * qw - 1) / (32 * qw)), tiles = (P.pos0 + P.n_rows + tk - 1) / tk;
    const size_t row = (size_t)P.n_rows * (P.dm.h * sizeof(float) + P.dm.H * sizeof(float2));
    const int parts = min(min(tiles / 2, (256 + wgs - 1) / wgs), min(kPfAttnPartsMax, (int)(P.part_bytes / row)));
    return parts >= 2 && tiles - (tiles + parts - 1) / parts >= 5 ? parts : 1;
}
template <int D, int QW, bool SPLIT>
static hipError_t pf_attention_launch(const PfParams &P, const PfAttnParts &A, hipStream_t s)
{
    constexpr int lds = pf_attn_lds<D, QW>();
    if constexpr (lds > 64 * 1024) {                       // (more than the default limit)
        const hipError_t e = hipFuncSetAttribute((const void *)k_pf_attn<D, QW, SPLIT, 0>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_pf_attn<D, QW, SPLIT, 0>), dim3(P.dm.H, A.blocks, A.parts), dim3(256), lds, s, P, A);
    return hipGetLastError();
}
template <int D, int QW>
static hipError_t pf_attention_of(const PfParams &P, hipStream_t s)
{
    const int blocks = (P.n_rows + 32 * QW - 1) / (32 * QW), wgs = P.dm.H * blocks;
    PfAttnParts A{P.part, nullptr, 1, blocks, 0};
    if constexpr (QW == (D == 128 ? 2 : 1)) {              // (with more queries to a workgroup there are more workgroups than CUs)
        A.parts = pf_attn_parts(P);
        if (A.parts > 1) A.ml = reinterpret_cast<float2 *>(P.part + (size_t)A.parts * P.n_rows * P.dm.h);
        A.first_down = wgs * A.parts;
        const bool down = P.nrw.on && P.nrw.downs > 0;
        if (down || A.parts > 1) {
            const hipError_t e = down ? launch_pf_attention_beside(P, A, s) : pf_attention_launch<D, QW, true>(P, A, s);
            if (e != hipSuccess || A.parts == 1) return e;
            hipLaunchKernelGGL(k_pf_attn_join<D>, dim3(P.dm.H, (P.n_rows + 31) / 32), dim3(256), 0, s, P, A);
            return hipGetLastError();
        }
    }
    return pf_attention_launch<D, QW, false>(P, A, s);
}
template <int D>
static hipError_t pf_attention(const PfParams &P, hipStream_t s)
{
    const int qw = pf_attn_blocks(P.dm, P.n_rows);
    if (qw == 4) return pf_attention_of<D, 4>(P, s);
    if (qw == 2) return pf_attention_of<D, 2>(P, s);
    if constexpr (D != 128) return pf_attention_of<D, 1>(P, s);
    return hipErrorInvalidValue;
}

template <bool FROM_PARTS>
static void pf_rows(const PfParams &P, hipStream_t s)
{
    if (P.n_rows <= kPfRowWide) hipLaunchKernelGGL((k_pf_row<FROM_PARTS, 1024>), dim3(P.n_rows), dim3(1024), 0, s, P);
    else hipLaunchKernelGGL((k_pf_row<FROM_PARTS, 256>), dim3(P.n_rows), dim3(256), 0, s, P);
}

hipError_t launch_pf_layer(const PfParams &P, hipStream_t s)
{
    const Dims &dm = P.dm;
    // (else the previous layer's last launch has left this one's input ready)
    if (P.layer == 0 || !P.row_fused) pf_rows<false>(P, s);
    hipError_t e = P.nrw.on ? launch_pf_narrow_in(P, s) : launch_pf_gemm_in(P, s);
    if (e != hipSuccess) return e;
    switch (dm.d) {
    case 64: e = pf_attention<64>(P, s); break;
    case 80: e = pf_attention<80>(P, s); break;
    case 128: e = pf_attention<128>(P, s); break;
    default: e = hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    e = P.nrw.on ? launch_pf_narrow_out(P, s) : launch_pf_gemm_out(P, s);
    if (e != hipSuccess) return e;
    if (P.plan_out.splits > 1 || P.nrw.on) pf_rows<true>(P, s);
    return hipGetLastError();
}

}  // namespace cfpp
