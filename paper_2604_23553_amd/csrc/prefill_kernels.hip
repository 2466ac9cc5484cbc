// Prompt processing with the weights read once per pass over up to kPfMaxRows
// tokens (the paper names a prefill phase beside its fused decode kernel, Sec. 4.2;
// what is computed is the block of Sec. 2.2 applied to every prompt token with
// causal attention).  With hundreds of tokens the four projections are dense
// contractions - tokens x K activations times K x rows weights - and run as
// LDS-tiled GEMMs on the matrix cores (prefill_gemm.hip); the attention of
// a pass reads the cache rows its own QKV launch appended.
//
//   k_pf_ln     : per token: mean, 1/sigma, and gamma_1 * x, gamma_2 * x as two fp16
//                 planes each (head + remainder: y = hi + lo to ~2^-22, so that the
//                 fp16 matrix instruction reproduces the fp32 product to rounding)
//   the products: prefill_gemm.hip - QKV and MLP-up in one launch, output projection and
//                 MLP-down as one product
//   k_pf_attn<> : causal attention of a block of 16 queries of one head over the cache,
//                 keys in LDS tiles of 64 positions, both products on the matrix
//                 cores (v_mfma_f32_16x16x16_f16), online softmax in fp32
//
// Every sum has a fixed order: one bit pattern per build and pass size.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "prefill_device.h"

namespace cfpp {

// ---------------------------------------------------------------------------
// One wavefront per scratch row, four rows per workgroup, no barrier: a lane holds the
// row's elements 4 (lane + 64 j) .. + 3, j < h / 256 (hidden: a multiple of 128, at most
// 4096; with an odd number of 128s the upper half of the lanes sits out the last j).
// Rows past the pass's tokens get zero planes (their products are never stored).
constexpr int kPfLnVec = 16;           // float4 per lane: hidden <= 4096
__global__ void __launch_bounds__(256) k_pf_ln(PfParams P)
{
    const Dims &dm = P.dm;
    const int h = dm.h, lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nv = h >> 2;                                 // groups of 4 elements in a row
    if (row >= P.n_rows) {
        const uint2 z = {0u, 0u};
        for (int g = lane; g < nv; g += 64) {
            const size_t at = pf_at(row, 4 * g, h);
            *reinterpret_cast<uint2 *>(P.y1 + at) = z; *reinterpret_cast<uint2 *>(P.y1 + at + kPfLo) = z;
            *reinterpret_cast<uint2 *>(P.y2 + at) = z; *reinterpret_cast<uint2 *>(P.y2 + at + kPfLo) = z;
        }
        return;
    }
    f32x4 x[kPfLnVec];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < kPfLnVec; ++j) {
        const int g = lane + 64 * j;
        x[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (g < nv) {
            if (P.layer == 0) {
                const uint2 w = *reinterpret_cast<const uint2 *>(P.x_in + (size_t)row * h + 4 * g);
                const float2 a = unpack_h2(w.x), b = unpack_h2(w.y);
                x[j] = f32x4{a.x, a.y, b.x, b.y};
                *reinterpret_cast<f32x4 *>(P.xres + (size_t)row * h + 4 * g) = x[j];
            } else {
                x[j] = *reinterpret_cast<const f32x4 *>(P.xres + (size_t)row * h + 4 * g);
            }
        }
        s += (x[j][0] + x[j][1]) + (x[j][2] + x[j][3]);
    }
    const float mean = wave_sum(s) / (float)h;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < kPfLnVec; ++j) {
        if (lane + 64 * j < nv) {
            const f32x4 dl = x[j] - mean;
            q += (dl[0] * dl[0] + dl[1] * dl[1]) + (dl[2] * dl[2] + dl[3] * dl[3]);
        }
    }
    const float inv = 1.0f / sqrtf(wave_sum(q) / (float)h + dm.ln_eps);
    if (lane == 0) P.stats[row] = float2{mean, inv};
    const __half *g1 = P.w + P.lay.ln1_g, *g2 = P.w + P.lay.ln2_g;
#pragma unroll
    for (int j = 0; j < kPfLnVec; ++j) {
        const int g = lane + 64 * j;
        if (g < nv) {
            const uint2 w1 = *reinterpret_cast<const uint2 *>(g1 + 4 * g), w2 = *reinterpret_cast<const uint2 *>(g2 + 4 * g);
            const float2 a1 = unpack_h2(w1.x), b1 = unpack_h2(w1.y), a2 = unpack_h2(w2.x), b2 = unpack_h2(w2.y);
            const float ga[4] = {a1.x, a1.y, b1.x, b1.y}, gb[4] = {a2.x, a2.y, b2.x, b2.y};
            __half h1[4], l1[4], h2[4], l2[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                pf_split(x[j][e] * ga[e], h1[e], l1[e]);
                pf_split(x[j][e] * gb[e], h2[e], l2[e]);
            }
            const size_t at = pf_at(row, 4 * g, h);
            *reinterpret_cast<uint2 *>(P.y1 + at) = *reinterpret_cast<const uint2 *>(h1);
            *reinterpret_cast<uint2 *>(P.y1 + at + kPfLo) = *reinterpret_cast<const uint2 *>(l1);
            *reinterpret_cast<uint2 *>(P.y2 + at) = *reinterpret_cast<const uint2 *>(h2);
            *reinterpret_cast<uint2 *>(P.y2 + at + kPfLo) = *reinterpret_cast<const uint2 *>(l2);
        }
    }
}

// ---------------------------------------------------------------------------
// Causal attention of kPfQB = 16 consecutive queries of one head: grid (H, blocks of
// queries), 4 wavefronts, on the matrix cores (v_mfma_f32_16x16x16_f16).  Keys and
// values of 64 positions at a time in LDS; wavefront w takes the tile's keys
// 16 w .. 16 w + 15:
//   S^T = K Q^T  (keys x queries): the instruction's result layout - a lane holds 4
//         consecutive keys of query lane % 16 - is at once the layout of the first
//         operand of the next product, so the weights never leave the registers;
//   O_w += P V   (queries x dimensions), P = exp(S - m) with the running maximum m of
//         the online softmax exchanged between the wavefronts through LDS once per
//         tile; V sits in LDS transposed ([dimension][key]) for that.
// q and P are fp32 values and enter as fp16 head + remainder (two instructions each),
// K and V are the cache's fp16; sums in fp32.  The wavefronts' partial outputs and
// partial softmax sums are added in wavefront order at the end.
constexpr int kPfQB = 16;
typedef _Float16 pf_f16x4 __attribute__((ext_vector_type(4)));

// maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the 16-lane rows of the wavefront)
__device__ __forceinline__ float pf_rows_max(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const unsigned u2 = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane32_swap(u2, u2, false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float pf_rows_sum(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const unsigned u2 = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane32_swap(u2, u2, false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// A tile of 64 cache positions x D dimensions of K and V on its way into LDS: pieces of 8 halves
// (one 16-byte load, slab by slab) held in registers from the request, one tile ahead of the
// arithmetic, to the store - K as rows [position][dimension], V transposed [dimension][position].
// Positions past `last_pos` repeat that row (the callers mask them).
template <int D>
struct PfKvTile {
    static constexpr int kPieces = 64 * (D / 8), kPer = (kPieces + 255) / 256;
    u32x4 k[kPer], v[kPer];
    __device__ __forceinline__ void request(const __half *Kc, const __half *Vc, int t0, int last_pos, int max_seq, int tid)
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = min(tid + 256 * i, kPieces - 1);
            const int pc = e / 64, t = e - pc * 64;        // piece pc = dims 8 pc .. 8 pc + 7 of position t0 + t
            const int tp = min(t0 + t, last_pos);
            const size_t off = ((size_t)(pc >> 1) * max_seq + tp) * 16 + (pc & 1) * 8;
            k[i] = load16(Kc + off);
            v[i] = load16(Vc + off);
        }
    }
    __device__ __forceinline__ void store(__half *sK, __half *sVt, int QS, int VS, int tid) const
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + 256 * i;
            if (e < kPieces) {
                const int pc = e / 64, t = e - pc * 64;
                unsigned *dk = reinterpret_cast<unsigned *>(&sK[t * QS + 8 * pc]);
                dk[0] = k[i].x; dk[1] = k[i].y; dk[2] = k[i].z; dk[3] = k[i].w;
                const __half *vh = reinterpret_cast<const __half *>(&v[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) sVt[(8 * pc + j) * VS + t] = vh[j];
            }
        }
    }
};

template <int D>
__global__ void __launch_bounds__(256) k_pf_attn(PfParams P)
{
    constexpr int QS = D + 4;                              // halves per row of q and K in LDS (8-byte fragment reads, spread over the banks)
    constexpr int VS = 64 + 4;                             // halves per row of V transposed
    constexpr int NB = D / 16;                             // 16-dimension blocks
    __shared__ __align__(16) __half sQh[kPfQB * QS], sQl[kPfQB * QS];
    constexpr int KVH = 64 * QS + D * VS;                  // halves of a tile of K and V
    static_assert(KVH * 2 >= 4 * kPfQB * D * 4 && (64 * QS) % 8 == 0, "the wavefronts' outputs reuse the tile's memory");
    __shared__ __align__(16) __half sKV[KVH];
    __shared__ float sMax[4][kPfQB], sCorr[4][kPfQB], sL[4][kPfQB];
    __half *sK = sKV, *sVt = sKV + 64 * QS;
    float (*sO)[kPfQB][D] = reinterpret_cast<float (*)[kPfQB][D]>(sKV);      // after the last tile
    const Dims &dm = P.dm;
    const int head = blockIdx.x, q0 = blockIdx.y * kPfQB, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q0 >= P.n_rows) return;
    const int nq = min(kPfQB, P.n_rows - q0);
    const float scale = 1.0f / sqrtf((float)D);
    for (int e = tid; e < kPfQB * D; e += 256) {
        const int qi = e / D, dmi = e - qi * D;
        const float v = qi < nq ? P.q[(size_t)(q0 + qi) * dm.h + head * D + dmi] * scale : 0.f;
        __half hi, lo;
        pf_split(v, hi, lo);
        sQh[qi * QS + dmi] = hi; sQl[qi * QS + dmi] = lo;
    }
    const int col = lane & 15, grp = lane >> 4;            // column of a result tile, group of 4 rows / 4 K values
    const int qpos = P.pos0 + q0 + col;                    // position of the query this lane's S^T column belongs to
    const bool qlive = col < nq;
    float m_run = -INFINITY, l_part = 0.f;                 // running maximum (all wavefronts alike), this wavefront's sum
    f32x4 O[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) O[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int last_pos = P.pos0 + q0 + nq - 1;             // the block's last query attends up to here
    const __half *Kc = P.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vc = P.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    PfKvTile<D> tile;
    tile.request(Kc, Vc, 0, last_pos, dm.max_seq, tid);
    for (int t0 = 0; t0 <= last_pos; t0 += 64) {
        __syncthreads();                                   // the previous tile is no longer read (first: q is written)
        tile.store(sK, sVt, QS, VS, tid);
        tile.request(Kc, Vc, t0 + 64, last_pos, dm.max_seq, tid);   // the next tile travels while this one is worked on
        __syncthreads();
        // S^T of this wavefront's 16 keys: rows = keys 16 wave + 4 grp + v, column = query col
        f32x4 st = {0.f, 0.f, 0.f, 0.f};
        const __half *ka = &sK[(16 * wave + col) * QS + 4 * grp];
        const __half *qh = &sQh[col * QS + 4 * grp], *ql = &sQl[col * QS + 4 * grp];
#pragma unroll
        for (int ks = 0; ks < NB; ++ks) {
            const pf_f16x4 kf = *reinterpret_cast<const pf_f16x4 *>(ka + 16 * ks);
            st = __builtin_amdgcn_mfma_f32_16x16x16f16(kf, *reinterpret_cast<const pf_f16x4 *>(qh + 16 * ks), st, 0, 0, 0);
            st = __builtin_amdgcn_mfma_f32_16x16x16f16(kf, *reinterpret_cast<const pf_f16x4 *>(ql + 16 * ks), st, 0, 0, 0);
        }
        const int key0 = t0 + 16 * wave + 4 * grp;
        float mloc = -INFINITY;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            st[v] = qlive && key0 + v <= qpos ? st[v] : -INFINITY;
            mloc = fmaxf(mloc, st[v]);
        }
        mloc = pf_rows_max(mloc);                          // over this wavefront's 16 keys, for query col
        if (lane < 16) sMax[wave][lane] = mloc;
        __syncthreads();
        const float mt = fmaxf(fmaxf(sMax[0][col], sMax[1][col]), fmaxf(sMax[2][col], sMax[3][col]));
        const float mn = fmaxf(m_run, mt);
        const float corr = m_run == -INFINITY ? 0.f : expf(m_run - mn);     // (mn finite whenever m_run is)
        float p[4], psum = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            p[v] = st[v] == -INFINITY ? 0.f : expf(st[v] - mn);
            psum += p[v];
        }
        l_part = l_part * corr + pf_rows_sum(psum);
        m_run = mn;
        if (lane < 16) sCorr[wave][lane] = corr;           // (read below by this wavefront only: no barrier)
        pf_f16x4 ph, pl;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const _Float16 h = (_Float16)p[v];
            ph[v] = h;
            pl[v] = (_Float16)(p[v] - (float)h);
        }
        // O rows = queries 4 grp + v, column = dimension 16 nb + col: rescale, then add P V of this wavefront's keys
        float cr[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) cr[v] = sCorr[wave][4 * grp + v];
        const __half *vb = &sVt[col * VS + 16 * wave + 4 * grp];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            f32x4 o = O[nb];
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] *= cr[v];
            const pf_f16x4 vf = *reinterpret_cast<const pf_f16x4 *>(vb + 16 * nb * VS);
            o = __builtin_amdgcn_mfma_f32_16x16x16f16(ph, vf, o, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f32_16x16x16f16(pl, vf, o, 0, 0, 0);
            O[nb] = o;
        }
    }
    // the wavefronts' parts, added in wavefront order
    __syncthreads();                                       // (the last tile is no longer read)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 4; ++v) sO[wave][4 * grp + v][16 * nb + col] = O[nb][v];
    if (lane < 16) sL[wave][lane] = l_part;
    __syncthreads();
    for (int e = tid; e < nq * D; e += 256) {
        const int qi = e / D, dmi = e - qi * D;
        const float l = ((sL[0][qi] + sL[1][qi]) + sL[2][qi]) + sL[3][qi];
        const float o = ((sO[0][qi][dmi] + sO[1][qi][dmi]) + sO[2][qi][dmi]) + sO[3][qi][dmi];
        __half hi, lo;
        pf_split(o / l, hi, lo);
        const size_t at = pf_at(q0 + qi, head * D + dmi, dm.h);
        P.o[at] = hi; P.o[at + kPfLo] = lo;
    }
}

// The same attention for long passes: 64 consecutive queries per workgroup, 16 per wavefront,
// every wavefront over all 64 keys of a tile.  A tile of K and V is then fetched once per 64
// queries instead of once per 16 (at 4096 tokens the narrow kernel pulls 10 GB per layer out of
// the L2), a wavefront's softmax is its own (no exchange between wavefronts), its q stays in
// registers as instruction operands, and a wavefront skips the tiles behind its last query.
// Blocks of later queries (more tiles) are started first.
constexpr int kPfQW = 64;
#ifndef PF_WIDE_FROM
#define PF_WIDE_FROM 1024
#endif
constexpr int kPfWideFrom = PF_WIDE_FROM;             // tokens in a pass from which the wide kernel runs

template <int D>
__global__ void __launch_bounds__(256) k_pf_attn_wide(PfParams P)
{
    constexpr int QS = D + 4, VS = 64 + 4, NB = D / 16;
    __shared__ __align__(16) __half sK[64 * QS];
    __shared__ __align__(16) __half sVt[D * VS];
    __shared__ float sX[4][16];                            // a per-query value from the lanes of the score layout to those of the output layout
    const Dims &dm = P.dm;
    const int head = blockIdx.x, q0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * kPfQW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q0 >= P.n_rows) return;
    const int nq = min(kPfQW, P.n_rows - q0);
    const float scale = 1.0f / sqrtf((float)D);
    const int col = lane & 15, grp = lane >> 4;
    const int qw0 = q0 + 16 * wave, qi = qw0 + col;        // this wavefront's first query, this lane's query in the score layout
    const bool qlive = qi < P.n_rows;
    const int qpos = P.pos0 + qi;
    const int wave_last = qw0 < P.n_rows ? P.pos0 + min(qw0 + 15, P.n_rows - 1) : -1;
    pf_f16x4 qh[NB], ql[NB];                               // Q^T fragments: dimensions 16 ks + 4 grp .. + 3 of query col
#pragma unroll
    for (int ks = 0; ks < NB; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v = qlive ? P.q[(size_t)qi * dm.h + head * D + 16 * ks + 4 * grp + j] * scale : 0.f;
            const _Float16 hi = (_Float16)v;
            qh[ks][j] = hi;
            ql[ks][j] = (_Float16)(v - (float)hi);
        }
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 O[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) O[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int last_pos = P.pos0 + q0 + nq - 1;
    const __half *Kc = P.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vc = P.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    PfKvTile<D> tile;
    tile.request(Kc, Vc, 0, last_pos, dm.max_seq, tid);
    for (int t0 = 0; t0 <= last_pos; t0 += 64) {
        __syncthreads();                                   // the previous tile is no longer read
        tile.store(sK, sVt, QS, VS, tid);
        tile.request(Kc, Vc, t0 + 64, last_pos, dm.max_seq, tid);   // the next tile travels while this one is worked on
        __syncthreads();
        if (t0 > wave_last) continue;                      // (whole wavefront; the barriers are above)
        // S^T of the tile's four key blocks: rows = keys 16 kb + 4 grp + v, column = query col
        f32x4 st[4];
        float mloc = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
            const __half *ka = &sK[(16 * kb + col) * QS + 4 * grp];
#pragma unroll
            for (int ks = 0; ks < NB; ++ks) {
                const pf_f16x4 kf = *reinterpret_cast<const pf_f16x4 *>(ka + 16 * ks);
                a = __builtin_amdgcn_mfma_f32_16x16x16f16(kf, qh[ks], a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x16f16(kf, ql[ks], a, 0, 0, 0);
            }
            const int key0 = t0 + 16 * kb + 4 * grp;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                a[v] = qlive && key0 + v <= qpos ? a[v] : -INFINITY;
                mloc = fmaxf(mloc, a[v]);
            }
            st[kb] = a;
        }
        mloc = pf_rows_max(mloc);                          // over the tile's 64 keys, for query col
        const float mn = fmaxf(m_run, mloc);
        const float corr = m_run == -INFINITY ? 0.f : expf(m_run - mn);
        float psum = 0.f;
        pf_f16x4 ph[4], pl[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float pv = st[kb][v] == -INFINITY ? 0.f : expf(st[kb][v] - mn);
                psum += pv;
                const _Float16 hi = (_Float16)pv;
                ph[kb][v] = hi;
                pl[kb][v] = (_Float16)(pv - (float)hi);
            }
        l_run = l_run * corr + pf_rows_sum(psum);
        m_run = mn;
        if (lane < 16) sX[wave][lane] = corr;              // (written and read by this wavefront only: no barrier)
        float cr[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) cr[v] = sX[wave][4 * grp + v];
        // O rows = queries 4 grp + v, column = dimension 16 nb + col
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            f32x4 o = O[nb];
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] *= cr[v];
            const __half *vb = &sVt[(16 * nb + col) * VS + 4 * grp];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const pf_f16x4 vf = *reinterpret_cast<const pf_f16x4 *>(vb + 16 * kb);
                o = __builtin_amdgcn_mfma_f32_16x16x16f16(ph[kb], vf, o, 0, 0, 0);
                o = __builtin_amdgcn_mfma_f32_16x16x16f16(pl[kb], vf, o, 0, 0, 0);
            }
            O[nb] = o;
        }
    }
    if (lane < 16) sX[wave][lane] = l_run;
    float lr[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) lr[v] = sX[wave][4 * grp + v];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int qo = qw0 + 4 * grp + v;
        if (qo < P.n_rows) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                __half hi, lo;
                pf_split(O[nb][v] / lr[v], hi, lo);
                const size_t at = pf_at(qo, head * D + 16 * nb + col, dm.h);
                P.o[at] = hi; P.o[at + kPfLo] = lo;
            }
        }
    }
}

// ---------------------------------------------------------------------------
bool pf_supported(const Dims &dm)
{
    return dm.h % kPfTile == 0 && dm.f % kPfTile == 0 && dm.h <= 256 * kPfLnVec && (dm.d == 64 || dm.d == 80 || dm.d == 128) &&
           !(dm.flags & kFlagSequentialResidual) && dm.r % 2 == 0;
}

hipError_t launch_pf_layer(const PfParams &P, hipStream_t s)
{
    const Dims &dm = P.dm;
    const int mt = (P.n_rows + kPfTile - 1) / kPfTile;
    hipLaunchKernelGGL(k_pf_ln, dim3(mt * kPfTile / 4), dim3(256), 0, s, P);
    hipError_t e = launch_pf_gemm_in(P, s);
    if (e != hipSuccess) return e;
    if (P.n_rows >= kPfWideFrom) {
        const dim3 ag(dm.H, (P.n_rows + kPfQW - 1) / kPfQW);
        switch (dm.d) {
        case 64: hipLaunchKernelGGL(k_pf_attn_wide<64>, ag, dim3(256), 0, s, P); break;
        case 80: hipLaunchKernelGGL(k_pf_attn_wide<80>, ag, dim3(256), 0, s, P); break;
        case 128: hipLaunchKernelGGL(k_pf_attn_wide<128>, ag, dim3(256), 0, s, P); break;
        default: return hipErrorInvalidValue;
        }
    } else {
        const dim3 ag(dm.H, (P.n_rows + kPfQB - 1) / kPfQB);
        switch (dm.d) {
        case 64: hipLaunchKernelGGL(k_pf_attn<64>, ag, dim3(256), 0, s, P); break;
        case 80: hipLaunchKernelGGL(k_pf_attn<80>, ag, dim3(256), 0, s, P); break;
        case 128: hipLaunchKernelGGL(k_pf_attn<128>, ag, dim3(256), 0, s, P); break;
        default: return hipErrorInvalidValue;
        }
    }
    e = launch_pf_gemm_out(P, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

}  // namespace cfpp
