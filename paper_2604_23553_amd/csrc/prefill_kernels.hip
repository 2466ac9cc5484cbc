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
//   k_pf_attn<> : causal attention of a block of 32, 64 or 128 queries of one head over the
//                 cache, keys in LDS tiles, both products on the matrix cores
//                 (v_mfma_f32_32x32x16_f16), online softmax in fp32
//
// Every sum has a fixed order: one bit pattern per build and pass size.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "prefill_device.h"

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

// ---------------------------------------------------------------------------
// Causal attention of 32 QW consecutive queries of one head: grid (H, blocks of queries, the
// last - longest - first), 4 wavefronts, both products on the matrix cores
// (v_mfma_f32_32x32x16_f16).  Wavefront w takes 32 queries (w % QW) and, of every tile of TK keys
// in LDS, 32 SUB keys (w / QW):
//   S^T = K Q^T  (keys x queries): a lane holds query lane % 32 and keys 8 g + 4 (lane / 32) .. + 3,
//         g < 4, so a query's softmax is lane arithmetic and one exchange with lane ^ 32, and
//         registers 8 m .. 8 m + 7 are, as they stand, a lane's 8 K values of the next product
//         if V's operand takes the same keys in the same order;
//   O^T += V^T P^T (dimensions x queries): the running sums are rescaled lane by lane, and only
//         when some query's maximum has moved; V sits in LDS transposed ([dimension][key]).
// q (scaled by log2 e / sqrt(D)) and P are fp32 values and enter as fp16 head + remainder (two
// instructions each), K and V are the cache's fp16; sums and softmax in fp32.  Keys behind a
// query are masked in the tiles that the diagonal crosses only.  With QW < 4 the wavefronts of
// the same queries keep a maximum and sums of their own and are added in wavefront order at the end.
// What bounds it: vector instructions (about 12 per score for the exponential, the sum and the two
// halves of P) beside 22 matrix instructions per 32 x 32 scores at D = 80, in equal parts.
typedef _Float16 pf_f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 pf_f16x8 __attribute__((ext_vector_type(8)));
typedef float pf_f32x16 __attribute__((ext_vector_type(16)));

// the value of lane ^ 32
__device__ __forceinline__ float pf_other_half(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float((threadIdx.x & 32) ? p[0] : p[1]);
}

// A tile of TK cache positions x D dimensions of K and V on its way into LDS: pieces of 8 halves
// held in registers from the request, one tile ahead of the arithmetic, to the store - K as rows
// [position][dimension], V transposed [dimension][position], two positions to a word.
// Positions past `last_pos` repeat that row (the callers mask them).
template <int D, int TK>
struct PfKvTile {
    static constexpr int kPieces = TK * (D / 8), kPer = (kPieces + 255) / 256, kPairs = kPieces / 2, kPerV = (kPairs + 255) / 256;
    u32x4 k[kPer], v[kPerV][2];
    __device__ __forceinline__ void request(const __half *Kc, const __half *Vc, int t0, int last_pos, int max_seq, int tid)
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = min(tid + 256 * i, kPieces - 1);
            const int pc = e / TK, t = min(t0 + e % TK, last_pos);         // piece pc = dims 8 pc .. 8 pc + 7
            k[i] = load16(Kc + ((size_t)(pc >> 1) * max_seq + t) * 16 + (pc & 1) * 8);
        }
#pragma unroll
        for (int i = 0; i < kPerV; ++i) {
            const int e = min(tid + 256 * i, kPairs - 1);
            const int pc = e / (TK / 2), t = t0 + 2 * (e % (TK / 2));
            const __half *p = Vc + (size_t)(pc >> 1) * max_seq * 16 + (pc & 1) * 8;
            v[i][0] = load16(p + (size_t)min(t, last_pos) * 16);
            v[i][1] = load16(p + (size_t)min(t + 1, last_pos) * 16);
        }
    }
    __device__ __forceinline__ void store(__half *sK, __half *sVt, int KS, int VS, int tid) const
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + 256 * i;
            if (kPieces % 256 == 0 || e < kPieces) *reinterpret_cast<u32x4 *>(&sK[(e % TK) * KS + 8 * (e / TK)]) = k[i];
        }
#pragma unroll
        for (int i = 0; i < kPerV; ++i) {
            const int e = tid + 256 * i;
            if (kPairs % 256 == 0 || e < kPairs) {
                unsigned *d = reinterpret_cast<unsigned *>(&sVt[8 * (e / (TK / 2)) * VS + 2 * (e % (TK / 2))]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d[(2 * j) * (VS / 2)] = __builtin_amdgcn_perm(v[i][1][j], v[i][0][j], 0x05040100u);
                    d[(2 * j + 1) * (VS / 2)] = __builtin_amdgcn_perm(v[i][1][j], v[i][0][j], 0x07060302u);
                }
            }
        }
    }
};

// One wavefront: the attention of one query (row of the pass) of one head, key by key in fp32, nothing behind the query read.
template <int D>
__device__ __forceinline__ void pf_attn_alone(const PfParams &P, const __half *Kc, const __half *Vc, int head, int row, int lane)
{
    constexpr int NE = (D + 63) / 64;                      // dimensions lane + 64 e
    const Dims &dm = P.dm;
    const float scale = 1.44269504088896340736f / sqrtf((float)D);
    size_t at[NE];
    float q[NE], o[NE], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int dim = min(lane + 64 * e, D - 1);
        at[e] = (size_t)(dim >> 4) * dm.max_seq * 16 + (dim & 15);
        q[e] = lane + 64 * e < D ? P.q[(size_t)row * dm.h + head * D + dim] * scale : 0.f;
        o[e] = 0.f;
    }
    for (int t = 0; t <= P.pos0 + row; ++t) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < NE; ++e) s = lane + 64 * e < D ? fmaf(q[e], __half2float(Kc[at[e] + (size_t)t * 16]), s) : s;
        s = wave_sum(s);
        const float mn = fmaxf(m, s), corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn), p = __builtin_amdgcn_exp2f(s - mn);
        m = mn;
        l = l * corr + p;
#pragma unroll
        for (int e = 0; e < NE; ++e) o[e] = fmaf(p, __half2float(Vc[at[e] + (size_t)t * 16]), o[e] * corr);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        if (lane + 64 * e >= D) continue;
        __half hi, lo;
        split_half(o[e] / l, hi, lo);
        const size_t to = pf_out_at(P, row, head * D + lane + 64 * e, dm.h);
        P.o[to] = hi; P.o[to + pf_out_lo(P)] = lo;
    }
}

// The end of a block of 32 QW queries of a head (256 threads): `sums` gives a query's unnormalised sums of 8 dimensions and
// its weight; the outputs go to the planes.
template <int D, int QW, class Sums>
__device__ __forceinline__ void pf_attn_finish(const PfParams &P, const __half *Kc, const __half *Vc, int head, int q0, int last_pos, int tid, Sums sums)
{
    __shared__ int sBad[32 * QW], sEnd[3];                 // queries whose output is not finite; any; the positions of pf_attn_alone's rule
    const Dims &dm = P.dm;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 32 * QW) sBad[tid] = 0;
    if (tid == 0) { sEnd[0] = 0; sEnd[1] = -1; sEnd[2] = 0x7fffffff; }
    __syncthreads();
    for (int e = tid; e < 32 * QW * (D / 8); e += 256) {
        const int q = e / (D / 8), c8 = 8 * (e - q * (D / 8));
        if (q0 + q >= P.n_rows) continue;
        f32x4 v[2];
        const float l = sums(q, c8, v);
        __half hi[8], lo[8];
        bool finite = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float va = v[0][j] / l, vb = v[1][j] / l;
            finite = finite && fabsf(va) < INFINITY && fabsf(vb) < INFINITY;
            split_half(va, hi[j], lo[j]);
            split_half(vb, hi[4 + j], lo[4 + j]);
        }
        const size_t at = pf_out_at(P, q0 + q, head * D + c8, dm.h);
        *reinterpret_cast<u32x4 *>(P.o + at) = *reinterpret_cast<const u32x4 *>(hi);
        *reinterpret_cast<u32x4 *>(P.o + at + pf_out_lo(P)) = *reinterpret_cast<const u32x4 *>(lo);
        if (!finite) { sBad[q] = 1; sEnd[0] = 1; }
    }
    // A masked key's weight is zero, and zero times an infinite or NaN V row of a later token of this block is NaN: such
    // queries are worked out once more, each alone.  Which: those ahead of the last position of the block whose V is not
    // finite, unless they see a V row that is finite nowhere (nothing of their output is).
    __syncthreads();
    if (!sEnd[0]) return;                                  // (uniform)
    const int first = P.pos0 + q0;
    if (first + tid <= last_pos) {                         // (a thread per position: 32 QW are at most 128)
        int bad = 0;
        for (int pc = 0; pc < D / 8; ++pc) {
            const u32x4 v = load16(Vc + ((size_t)(pc >> 1) * dm.max_seq + first + tid) * 16 + (pc & 1) * 8);
#pragma unroll
            for (int j = 0; j < 4; ++j) bad += ((v[j] & 0x7c00u) == 0x7c00u) + ((v[j] & 0x7c000000u) == 0x7c000000u);
        }
        if (bad) atomicMax(&sEnd[1], first + tid);
        if (bad == D) atomicMin(&sEnd[2], first + tid);
    }
    __syncthreads();
    const int end = min(sEnd[1], sEnd[2]);
    for (int q = wave; q < 32 * QW && first + q < end; q += 4)         // (a query ahead of a position of the block is one of the pass)
        if (sBad[q]) pf_attn_alone<D>(P, Kc, Vc, head, q0 + q, lane);
}

// SPLIT: workgroup z of a head's block takes the z-th part of the block's tiles of keys and leaves its queries' sums,
// maxima and weights in memory, where k_pf_attn_join adds them.  For few queries behind a long context: a workgroup takes a
// tile of keys in about 1.3 us, and 37 queries of 32 heads are 64 workgroups.
template <int D, int QW, bool SPLIT>
__global__ void __launch_bounds__(256, 2) k_pf_attn(PfParams P, PfAttnParts A)
{
    constexpr int KW = 4 / QW, SUB = QW == 4 ? 2 : 1, TK = 32 * KW * SUB;
    constexpr int NK = D / 16, NB = (D + 31) / 32;         // K steps of S, 32-dimension tiles of O
    constexpr int KS = D + 8, VS = TK + 4;                 // halves per row of K and of V transposed: fragment reads spread over all banks
    constexpr int OS = D + 4;                              // floats per query of a wavefront's output in LDS
    constexpr int kTileBytes = (TK * KS + 32 * NB * VS) * 2, kOutBytes = 4 * 32 * OS * 4;
    __shared__ __align__(16) char mem[kTileBytes > kOutBytes ? kTileBytes : kOutBytes];
    __shared__ float sM[4][32], sL[4][32];
    __half *sK = reinterpret_cast<__half *>(mem), *sVt = sK + TK * KS;
    static_assert((TK * KS * 2) % 16 == 0, "");
    const Dims &dm = P.dm;
    const int head = blockIdx.x, q0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * 32 * QW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (q0 >= P.n_rows) return;
    const int wq = wave % QW, wk = wave / QW, col = lane & 31, hf = lane >> 5;
    const int qw0 = q0 + 32 * wq, qi = qw0 + col;          // this wavefront's first query, this lane's
    const int qpos = P.pos0 + qi, first_pos = P.pos0 + qw0;
    const int wave_last = qw0 < P.n_rows ? P.pos0 + min(qw0 + 31, P.n_rows - 1) : -1;
    const int last_pos = P.pos0 + min(q0 + 32 * QW, P.n_rows) - 1;         // the block's last query attends up to here
    const __half *Kc = P.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vc = P.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    const int tiles = (last_pos + TK) / TK;                // (last_pos / TK + 1)
    const int t_first = SPLIT ? tiles * (int)blockIdx.z / A.parts * TK : 0, t_end = SPLIT ? tiles * ((int)blockIdx.z + 1) / A.parts * TK : tiles * TK;
    PfKvTile<D, TK> tile;
    tile.request(Kc, Vc, t_first, last_pos, dm.max_seq, tid);
    pf_f16x8 qh[NK], ql[NK];                               // Q^T: dimensions 16 ks + 8 hf .. + 7 of query col
    const float scale = 1.44269504088896340736f / sqrtf((float)D);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        // (a lane without a query takes the last one's: its results are not stored)
        const f32x4 *qp = reinterpret_cast<const f32x4 *>(P.q + (size_t)min(qi, P.n_rows - 1) * dm.h + head * D + 16 * ks + 8 * hf);
        const f32x4 a = qp[0], b = qp[1];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float v = split_value((j < 4 ? a[j & 3] : b[j & 3]) * scale);
            qh[ks][j] = (_Float16)v;
            ql[ks][j] = (_Float16)(v - (float)qh[ks][j]);
        }
    }
    float m_run = -INFINITY, l_run = 0.f;                  // l_run: of this lane's keys
    pf_f32x16 O[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[nb][e] = 0.f;
    for (int t0 = t_first; t0 < t_end; t0 += TK) {
        __syncthreads();                                   // the previous tile is no longer read
        tile.store(sK, sVt, KS, VS, tid);
        tile.request(Kc, Vc, t0 + TK, last_pos, dm.max_seq, tid);      // the next tile travels while this one is worked on
        __syncthreads();
        const int kw0 = 32 * SUB * wk;                     // this wavefront's first key in the tile
        if (t0 + kw0 > wave_last) continue;                // (whole wavefront; the barriers are above)
        pf_f32x16 st[SUB];
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) st[s][e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            pf_f16x8 kf[SUB];
#pragma unroll
            for (int s = 0; s < SUB; ++s) kf[s] = *reinterpret_cast<const pf_f16x8 *>(&sK[(kw0 + 32 * s + col) * KS + 16 * ks + 8 * hf]);
#pragma unroll
            for (int s = 0; s < SUB; ++s) st[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s], qh[ks], st[s], 0, 0, 0);
#pragma unroll
            for (int s = 0; s < SUB; ++s) st[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s], ql[ks], st[s], 0, 0, 0);
        }
        if (t0 + kw0 + 32 * SUB - 1 > first_pos) {         // (uniform) the diagonal is not behind every key
#pragma unroll
            for (int s = 0; s < SUB; ++s)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (t0 + kw0 + 32 * s + 8 * (e >> 2) + 4 * hf + (e & 3) > qpos) st[s][e] = -INFINITY;
        }
        float mloc = st[0][0];
#pragma unroll
        for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) mloc = fmaxf(mloc, st[s][e]);
        mloc = fmaxf(mloc, pf_other_half(mloc));
        if (__any(mloc > m_run)) {                         // (uniform) some query's maximum moves
            const float mn = fmaxf(m_run, mloc);
            const float corr = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mn);
            m_run = mn;
            l_run *= corr;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) O[nb][e] *= corr;
        }
        const float mref = m_run == -INFINITY ? 0.f : m_run;           // (a query none of whose keys this wavefront has seen)
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
            pf_f16x8 ph[2], pl[2];
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float p = __builtin_amdgcn_exp2f(st[s][e] - mref);
                sum += p;
                const _Float16 h = (_Float16)p;
                ph[e >> 3][e & 7] = h;
                pl[e >> 3][e & 7] = (_Float16)(p - (float)h);
            }
            l_run += sum;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const __half *vp = &sVt[(32 * nb + col) * VS + kw0 + 32 * s + 16 * m + 4 * hf];
                    const pf_f16x4 v0 = *reinterpret_cast<const pf_f16x4 *>(vp), v1 = *reinterpret_cast<const pf_f16x4 *>(vp + 8);
                    const pf_f16x8 vf = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                    O[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, ph[m], O[nb], 0, 0, 0);
                    O[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pl[m], O[nb], 0, 0, 0);
                }
        }
    }
    // the outputs through LDS (a query's dimensions side by side), where wavefronts of the same queries meet
    l_run += pf_other_half(l_run);
    float corr = 1.f;
    if (KW > 1 || SPLIT) {
        if (hf == 0) { sM[wave][col] = m_run; }
        __syncthreads();
    }
    if (KW > 1) {
        float m = sM[wq][col];
#pragma unroll
        for (int w = 1; w < KW; ++w) m = fmaxf(m, sM[wq + QW * w][col]);
        corr = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m);
    }
    if (hf == 0) sL[wave][col] = l_run * corr;
    __syncthreads();                                       // (the last tile is no longer read)
    float *out = reinterpret_cast<float *>(mem) + (wave * 32 + col) * OS;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int dim = 32 * nb + 8 * g + 4 * hf;
            if (32 * nb + 8 * g < D)
                *reinterpret_cast<f32x4 *>(out + dim) = f32x4{O[nb][4 * g] * corr, O[nb][4 * g + 1] * corr, O[nb][4 * g + 2] * corr, O[nb][4 * g + 3] * corr};
        }
    __syncthreads();
    const float *res = reinterpret_cast<const float *>(mem);
    // what the block's wavefronts have of query q, dimensions c8 .. + 7: unnormalised sums and weight
    auto sums = [&](int q, int c8, f32x4 (&v)[2]) {
        const int w0 = q >> 5, qc = q & 31;
        float l = sL[w0][qc];
        v[0] = *reinterpret_cast<const f32x4 *>(res + (w0 * 32 + qc) * OS + c8); v[1] = *reinterpret_cast<const f32x4 *>(res + (w0 * 32 + qc) * OS + c8 + 4);
#pragma unroll
        for (int w = 1; w < KW; ++w) {
            const int ww = w0 + QW * w;
            l += sL[ww][qc];
            v[0] += *reinterpret_cast<const f32x4 *>(res + (ww * 32 + qc) * OS + c8);
            v[1] += *reinterpret_cast<const f32x4 *>(res + (ww * 32 + qc) * OS + c8 + 4);
        }
        return l;
    };
    if (SPLIT) {
        for (int e = tid; e < 32 * QW * (D / 8); e += 256) {
            const int q = e / (D / 8), c8 = 8 * (e - q * (D / 8));
            if (q0 + q >= P.n_rows) continue;
            f32x4 v[2];
            const float l = sums(q, c8, v);
            const size_t row = (size_t)blockIdx.z * P.n_rows + q0 + q;
            f32x4 *o = reinterpret_cast<f32x4 *>(A.o + row * dm.h + head * D + c8);
            o[0] = v[0]; o[1] = v[1];
            if (c8 == 0) {
                float m = sM[q >> 5][q & 31];
#pragma unroll
                for (int w = 1; w < KW; ++w) m = fmaxf(m, sM[(q >> 5) + QW * w][q & 31]);
                A.ml[row * dm.H + head] = float2{m, l};
            }
        }
        return;
    }
    pf_attn_finish<D, QW>(P, Kc, Vc, head, q0, last_pos, tid, sums);
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
template <int D, int QW>
static void pf_attention_of(const PfParams &P, hipStream_t s)
{
    constexpr int TK = 128 / QW * (QW == 4 ? 2 : 1);
    const int blocks = (P.n_rows + 32 * QW - 1) / (32 * QW), wgs = P.dm.H * blocks, tiles = (P.pos0 + P.n_rows + TK - 1) / TK;
    PfAttnParts A{P.part, nullptr, 1};
    if constexpr (QW == (D == 128 ? 2 : 1)) {              // (with more queries to a workgroup there are more workgroups than CUs)
        const size_t row = (size_t)P.n_rows * (P.dm.h * sizeof(float) + P.dm.H * sizeof(float2));
        const int parts = min(min(tiles / 2, (256 + wgs - 1) / wgs), min(kPfAttnPartsMax, (int)(P.part_bytes / row)));
        if (parts >= 2 && tiles - (tiles + parts - 1) / parts >= 5) {
            A.parts = parts;
            A.ml = reinterpret_cast<float2 *>(P.part + (size_t)parts * P.n_rows * P.dm.h);
            hipLaunchKernelGGL((k_pf_attn<D, QW, true>), dim3(P.dm.H, blocks, parts), dim3(256), 0, s, P, A);
            hipLaunchKernelGGL(k_pf_attn_join<D>, dim3(P.dm.H, (P.n_rows + 31) / 32), dim3(256), 0, s, P, A);
            return;
        }
    }
    hipLaunchKernelGGL((k_pf_attn<D, QW, false>), dim3(P.dm.H, blocks), dim3(256), 0, s, P, A);
}
template <int D>
static void pf_attention(const PfParams &P, hipStream_t s)
{
    const int n = P.dm.H * ((P.n_rows + 31) / 32);
    const int qw = n >= (D == 128 ? 1536 : 2048) ? 4 : D == 128 || n >= 768 ? 2 : 1;
    if (qw == 4) pf_attention_of<D, 4>(P, s);
    else if (qw == 2) pf_attention_of<D, 2>(P, s);
    else if constexpr (D != 128) pf_attention_of<D, 1>(P, s);
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
    case 64: pf_attention<64>(P, s); break;
    case 80: pf_attention<80>(P, s); break;
    case 128: pf_attention<128>(P, s); break;
    default: return hipErrorInvalidValue;
    }
    e = P.nrw.on ? launch_pf_narrow_out(P, s) : launch_pf_gemm_out(P, s);
    if (e != hipSuccess) return e;
    if (P.plan_out.splits > 1 || P.nrw.on) pf_rows<true>(P, s);
    return hipGetLastError();
}

}  // namespace cfpp
