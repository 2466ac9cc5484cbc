// Causal attention of the prompt-sized path (launched by prefill_kernels.hip and, with MLP-down beside it, prefill_beside.hip).
#pragma once
#include "narrow_stream.h"
#include "prefill_device.h"

namespace cfpp {

// Causal attention of 32 QW consecutive queries of one head: grid (H, blocks of queries, the
// last - longest - first), 4 wavefronts, both products on the matrix cores
// (v_mfma_f32_32x32x16_f16).  Wavefront w takes 32 queries (w % QW) and, of every tile of TK keys
// in LDS, 32 SUB keys (w / QW):
//   S^T = K Q^T  (keys x queries): a lane holds query lane % 32 and keys 8 g + 4 (lane / 32) .. + 3,
//         g < 4, so a query's softmax is lane arithmetic and one exchange with lane ^ 32, and
//         registers 8 m .. 8 m + 7 are, as they stand, a lane's 8 K values of the next product
//         if V's operand takes the same keys in the same order;
//   O^T += V^T P^T (dimensions x queries): the running sums are rescaled lane by lane, and only
//         when some query's maximum has moved by more than 2^4 (kPfFollow); V sits in LDS transposed ([dimension][key]).
// q (scaled by log2 e / sqrt(D)) and P are fp32 values and enter as fp16 head + remainder (two
// instructions each), K and V are the cache's fp16; sums and softmax in fp32.  Keys behind a
// query are masked in the tiles that the diagonal crosses only.  With QW < 4 the wavefronts of
// the same queries keep a maximum and sums of their own and are added in wavefront order at the end.
// What bounds it: vector instructions (about 7 per score: difference, exponential, sum, maximum, the two halves of P) beside 22 matrix
// instructions per 32 x 32 scores at D = 80, in equal parts.  Two halves of P come from one conversion and a remainder from one v_fma_mix;
// with a reference that follows a query's maximum only when it has to, 8.3 -> 7.2 vector instructions a score.
// The scores' sums start at zero and the reference is subtracted behind them.  Starting them at minus the reference would save the subtraction,
// but where a query's scores then rise by J its sums carry roundings of the size of J: error of the outputs against 64 bits after a
// rise of 30 / 500 / 2000 in base 2, D = 64: 4.7e-7 / 7.5e-6 / 2.7e-5, as it is 5.3e-8 / 4.1e-8 / 4.1e-8 (80 and 128 alike), and at no size measured
// was it more than 1 % faster.  Where nothing rises a large score's last sums then end near zero, and its roundings are a quarter smaller (queries and keys
// six times as large, D = 64 / 80 / 128: 4.7e-7 / 1.2e-6 / 1.8e-6, as it is 6.6e-7 / 1.5e-6 / 2.3e-6).  Adding all remainders ahead of the heads does that too, at any
// rise (4.8e-7 / 1.1e-6 / 1.6e-6), for 0.3 - 0.7 % of a layer at 1500 tokens and more; not taken.
typedef _Float16 pf_f16x2 __attribute__((ext_vector_type(2)));
typedef float pf_f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 pf_f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 pf_f16x8 __attribute__((ext_vector_type(8)));
typedef float pf_f32x16 __attribute__((ext_vector_type(16)));

// p - h, exactly (minus_one: one that the compiler does not see through: it would convert h and subtract, two instructions for one)
__device__ __forceinline__ pf_f32x2 pf_remainder(pf_f32x2 p, pf_f16x2 h, float minus_one)
{
    return pf_f32x2{fmaf((float)h[0], minus_one, p[0]), fmaf((float)h[1], minus_one, p[1])};
}

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

// bytes of a tile of K and V, or of a block's outputs, in LDS
template <int D, int QW>
constexpr int pf_attn_lds()
{
    constexpr int TK = 128 / QW * (QW == 4 ? 2 : 1), tile = (TK * (D + 8) + 32 * ((D + 31) / 32) * (TK + 4)) * 2, out = 4 * 32 * (D + 4) * 4;
    return tile > out ? tile : out;
}

// MLP-down of a short prompt beside the attention (which it does not depend on): workgroup `id` has the rows of one group (16 T) and one
// part of K, each of its wavefronts a quarter of that, streamed as in narrow_stream.h; the parts are added where the next
// layer's input is made, together with the output projection's (k_pf_row).  Which passes take it, and what it gives: pf_down_parts.
template <int S>
constexpr int pf_down_tiles() { return S <= 5 ? 4 : 2; }               // two workgroups' rings to a CU
template <int S>
constexpr int pf_down_lds() { return 4 * NgStream<pf_down_tiles<S>(), S, kNgPlanes, 1>::kStage; }
template <int S>
__device__ __forceinline__ void pf_down(const PfParams &P, int id, char *lds)
{
    constexpr int T = pf_down_tiles<S>(), W = 4, ROWS = 16 * T;
    using Stream = NgStream<T, S, kNgPlanes, 1>;
    static_assert(W * S * Stream::kSetFloats * 4 <= pf_down_lds<S>(), "");
    const int h = P.dm.h, f = P.dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = id / P.nrw.downs, z = id - g * P.nrw.downs, r0 = g * ROWS;             // (hidden: a multiple of 128)
    const int C = f / kNgChunk, z0 = C * z / P.nrw.downs, zn = C * (z + 1) / P.nrw.downs - z0, c0 = z0 + zn * wave / W;
    Stream st;
    st.p0.w = P.w + P.lay.w_down + (size_t)r0 * f; st.p0.row_bytes = (unsigned)f * 2u;
    st.p0.b = P.m; st.p0.set_bytes = (unsigned)f * 32u; st.p0.b_bytes = S * st.p0.set_bytes;
    st.p0.c0 = c0; st.p0.n = z0 + zn * (wave + 1) / W - c0;
    st.p1 = st.p0; st.p1.n = 0;
    st.ring = lds_address(lds) + (unsigned)(wave * Stream::kStage);
    st.mem = lds + wave * Stream::kStage;
    st.gamma = nullptr;
    st.begin(ROWS, P.n_rows, kNgSet, 0u, tid);
    st.run();
    float *red = reinterpret_cast<float *>(lds), *part = P.part_out + (size_t)z * P.part_out_stride + r0;
    __syncthreads();                                       // the rings have been read
    st.template leave<S>(red, wave, 0);
    __syncthreads();
    for (int i = tid; i < P.n_rows * (ROWS / 2); i += 64 * W) {        // items of two rows of a token, a token's side by side
        const int token = i / (ROWS / 2), pr = i % (ROWS / 2);
        const float2 v = ng_total2<W>(red + (token >> 3) * Stream::kSetFloats, S * Stream::kSetFloats, 2 * pr, token & 7);
        *reinterpret_cast<float2 *>(part + (unsigned)(token * h + 2 * pr)) = v;
    }
}

// SPLIT: workgroup z of a head's block takes the z-th part of the block's tiles of keys and leaves its queries' sums,
// maxima and weights in memory, where k_pf_attn_join adds them.  For few queries behind a long context: a workgroup takes a
// tile of keys in about 1.3 us, and 37 queries of 32 heads are 64 workgroups.
// S > 0 (short prompts): workgroups behind the attention's have parts of MLP-down, S sets of 8 tokens (pf_down); one-dimensional grid.
template <int D, int QW, bool SPLIT, int S>
__global__ void __launch_bounds__(256, 2) k_pf_attn(PfParams P, PfAttnParts A)
{
    extern __shared__ __align__(16) char pf_mem[];
    int head = blockIdx.x, block = blockIdx.y, part = blockIdx.z;
    if constexpr (S > 0) {
        const int i = (int)blockIdx.x;
        if (i >= A.first_down) {
            pf_down<S>(P, i - A.first_down, pf_mem);
            return;
        }
        part = i / (P.dm.H * A.blocks);
        block = i / P.dm.H - part * A.blocks;
        head = i % P.dm.H;
    }
    constexpr int KW = 4 / QW, SUB = QW == 4 ? 2 : 1, TK = 32 * KW * SUB;
    constexpr int NK = D / 16, NB = (D + 31) / 32;         // K steps of S, 32-dimension tiles of O
    constexpr int KS = D + 8, VS = TK + 4;                 // halves per row of K and of V transposed: fragment reads spread over all banks
    constexpr int OS = D + 4;                              // floats per query of a wavefront's output in LDS
    constexpr int kTileBytes = (TK * KS + 32 * NB * VS) * 2, kOutBytes = 4 * 32 * OS * 4;
    static_assert(pf_attn_lds<D, QW>() == (kTileBytes > kOutBytes ? kTileBytes : kOutBytes), "");
    char *mem = pf_mem;
    __shared__ float sM[4][32], sL[4][32];
    __half *sK = reinterpret_cast<__half *>(mem), *sVt = sK + TK * KS;
    static_assert((TK * KS * 2) % 16 == 0, "");
    const Dims &dm = P.dm;
    const int q0 = (A.blocks - 1 - block) * 32 * QW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (q0 >= P.n_rows) return;
    const int wq = wave % QW, wk = wave / QW, col = lane & 31, hf = lane >> 5;
    const int qw0 = q0 + 32 * wq, qi = qw0 + col;          // this wavefront's first query, this lane's
    const int qpos = P.pos0 + qi, first_pos = P.pos0 + qw0;
    const int wave_last = qw0 < P.n_rows ? P.pos0 + min(qw0 + 31, P.n_rows - 1) : -1;
    const int last_pos = P.pos0 + min(q0 + 32 * QW, P.n_rows) - 1;         // the block's last query attends up to here
    const __half *Kc = P.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vc = P.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    const int tiles = (last_pos + TK) / TK;                // (last_pos / TK + 1)
    const int t_first = SPLIT ? tiles * part / A.parts * TK : 0, t_end = SPLIT ? tiles * (part + 1) / A.parts * TK : tiles * TK;
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
    // what the query's weights are relative to: its maximum or up to kPfFollow less (in base 2: the difference of two scores keeps its bits, and
    // the weights stay below 2^4); l_run: of this lane's keys.  us of layers with 1 / 4 / 8: hidden 512, 4000 tokens 1252 / 1246 / 1254,
    // 2560, 300 behind 3000 1615 / 1600 / 1596; with 8 the error after rises of 5 .. 8 is up to 11 % more in its largest, with 4 as with 0.
    constexpr float kPfFollow = 4.f;
    float m_run = -INFINITY, l_run = 0.f;
    pf_f32x16 O[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[nb][e] = 0.f;
    float minus_one = -1.f;
    asm("" : "+s"(minus_one));
    for (int t0 = t_first; t0 < t_end; t0 += TK) {
        __syncthreads();                                   // the previous tile is no longer read
        tile.store(sK, sVt, KS, VS, tid);
        tile.request(Kc, Vc, t0 + TK, last_pos, dm.max_seq, tid);      // the next tile travels while this one is worked on
        __syncthreads();
        const int kw0 = 32 * SUB * wk;                     // this wavefront's first key in the tile
        if (t0 + kw0 > wave_last) continue;                // (whole wavefront; the barriers are above)
        pf_f32x16 st[SUB];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            pf_f16x8 kf[SUB];
#pragma unroll
            for (int s = 0; s < SUB; ++s) kf[s] = *reinterpret_cast<const pf_f16x8 *>(&sK[(kw0 + 32 * s + col) * KS + 16 * ks + 8 * hf]);
#pragma unroll
            for (int s = 0; s < SUB; ++s) st[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s], qh[ks], ks ? st[s] : pf_f32x16{}, 0, 0, 0);
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
        // the query's first keys, or a score above what its weights are relative to by more than kPfFollow
        const bool moves = mloc > (m_run == -INFINITY ? -INFINITY : m_run + kPfFollow);
        if (__any(moves)) {                                // (uniform)
            const float corr = !moves ? 1.f : m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mloc);
            if (moves) m_run = mloc;
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
            for (int e = 0; e < 16; e += 2) {
                const pf_f32x2 p{__builtin_amdgcn_exp2f(st[s][e] - mref), __builtin_amdgcn_exp2f(st[s][e + 1] - mref)};
                sum += p[0];
                sum += p[1];
                const pf_f16x2 h = __builtin_convertvector(p, pf_f16x2);
                const pf_f32x2 r = pf_remainder(p, h, minus_one);
                const pf_f16x2 l = __builtin_convertvector(r, pf_f16x2);
                ph[e >> 3][e & 7] = h[0]; ph[e >> 3][(e & 7) + 1] = h[1];
                pl[e >> 3][e & 7] = l[0]; pl[e >> 3][(e & 7) + 1] = l[1];
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
            const size_t row = (size_t)part * P.n_rows + q0 + q;
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

}  // namespace cfpp
