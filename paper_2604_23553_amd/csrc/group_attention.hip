// Attention of a group of prompt tokens (2 .. 8 consecutive positions of one sequence, batched path) behind a longer context, and MLP-down in the same launch.
//
// The queries of a head read the same cached rows, so a workgroup takes them together: a piece of the positions ahead of the
// group, of one head, on the matrix cores (v_mfma_f32_16x16x32_f16).  A query's element or a weight goes in as two fp16 values, its head and
// 2^11 times what the head leaves: columns 0 .. 7 of an operand are the heads of the 8 queries, columns 8 .. 15 the others, and so are the sums:
//   S = K Q^T   (16 positions x 16 columns): a lane holds column lane % 16 and positions 4 (lane / 16) .. + 3; the two columns of a query are
//               eight lanes apart.  A query is scaled by a power of two first, its largest element to 2^14 .. 2^15, and its scores back.
//   O^T += V^T P^T (16 dimensions x 16 columns): a lane's 8 K values are the positions of its own scores in two tiles of 16, so that P
//               needs no exchange.  Weights go in 2^14 times.  V goes through LDS of the wavefront's own, transposed, two positions to a word.
// So an element or weight keeps 2^-23 of itself down to 2^-26 of the largest, and below that 2^-50 of the largest (the two as they are, half_split.h: 2^-25).
// Error of the outputs against 64 bits (2-norm; 8 tokens behind 1001 positions; head size 64 / 80 / 128), every query for itself in fp32 -> head
// and remainder as they are -> this:
//   queries four times as large as usual 7.5e-8 / 2.1e-7 / 2.6e-7 -> 6.8e-8 / 1.9e-7 / 3.2e-7 -> 6.5e-8 / 1.8e-7 / 2.6e-7;
//   light keys behind one of 2^16 times their weight, whose V is zero 1.4e-6 -> 7.5e-6 -> 1.4e-6 at all three;
//   a query's element of 3000 that meets zeros in K 2.2e-8 / 2.3e-8 / 2.4e-8 -> 3.1e-6 / 3.6e-6 / 4.2e-6 -> 2.2e-8 / 2.3e-8 / 2.5e-8.
// us of layers, head and remainder as they are -> this, 8 tokens: 32 of hidden 2560 behind 1000 1315 -> 1321, 10 of 4096 behind 3000 841 -> 837, 16 of 512
// behind 2500 291.2 -> 290.9.
// Every query sees every one of these positions.  The group's own rows, where the causal mask lies, are a workgroup more to a
// head, in fp32: no masked weight is ever multiplied by a V row.  An output that is not finite (a cached K or V element may be infinite, and
// what a head leaves zero) is worked out once more in fp32.
// Maxima and sums of the wavefronts and pieces are joined in order, as in narrow_attention.hip.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "attention_common.h"
#include "mlp_down.h"

namespace cfpp {

typedef _Float16 ga_f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 ga_f16x4 __attribute__((ext_vector_type(4)));

constexpr int kGaWaves = kAttnBatchThreads / 64, kGaRow = 32;          // positions of a row, a wavefront's step
constexpr int kGaStride = kGaRow + 4;                                  // halves between V's dimensions in LDS

// Pieces of the positions ahead of the group: about a row to each wavefront or more (a piece of three leaves one without), as many as fill the CUs once, and at most eight: with the
// group's own rows their sums are one round of loads (12 or 16 pieces, two rounds: hidden 1280 behind 2500 positions 26.1 -> 27.9 / 28.4 us a layer).  The group's own rows are a piece too: with 8 and that one 32
// heads are 288 workgroups, with 7 256: 8 tokens behind 1000 of hidden 2560 41.7 -> 41.2, of 4096 behind 3000 87.9 -> 84.2; with 5 or 6 0.5 .. 3.5 % more.
constexpr int kGaPieces = 8;
CFPP_HD int ga_pieces(int first, int H)
{
    const int rows = (first + kGaRow - 1) / kGaRow, want = (rows + kGaWaves - 1) / kGaWaves, fill = 256 / H - 1;
    const int n = want < fill ? want : fill < 1 ? 1 : fill;
    return n < kGaPieces ? n : kGaPieces;
}
// Where it is taken.  Below some 900 positions the pieces' way to memory and back (4 - 5 us, whatever their size) is more than the
// other kernel's reading of every row once a query.  16 .. 21 heads are 144 .. 189 workgroups, which leave that many of the 256 CUs without, and the
// other kernel nearly fills them: there heads x tokens x positions have to come to 160000.  us a layer, one query to a workgroup -> this, positions
// behind which 2 / 3 / 5 / 8 tokens attend:
//   8 heads of 64, hidden 512: 850 16.6 / 16.6 / 16.9 / 17.2 -> 15.7 / 15.8 / 16.8 / 17.2, 1000 16.5 / 16.6 / 17.2 / 17.5 -> 15.8 / 15.9 / 17.0 / 17.4, 4000 17.7 / 17.9 / 19.1 / 20.0 -> 17.7 / 17.8 / 18.8 / 19.1;
//   16 of 64, 1024: 1000 18.3 / 18.4 / 18.8 / 19.2 -> 18.6 / 18.8 / 19.9 / 20.2, 2000 18.8 / 18.8 / 20.5 / 21.5 -> 19.3 / 19.5 / 20.6 / 20.8, 4000 21.6 / 22.0 / 23.6 / 26.2 -> 22.2 / 22.3 / 23.4 / 23.7;
//   16 of 80, 1280: 1000 21.6 / 21.6 / 22.3 / 22.7 -> 21.3 / 21.4 / 22.6 / 24.1, 1500 21.9 / 22.7 / 23.9 / 24.4 -> 22.1 / 22.3 / 23.5 / 24.9, 3000 23.6 / 24.0 / 25.4 / 27.8 -> 23.6 / 23.8 / 25.1 / 26.7;
//   20 of 128, 2560: 1000 36.6 / 37.0 / 40.2 / 44.5 -> 38.4 / 39.0 / 40.3 / 42.5, 2000 39.0 / 40.7 / 45.6 / 52.6 -> 39.9 / 41.0 / 42.5 / 44.9, 3500 42.6 / 45.5 / 52.6 / 66.3 -> 43.4 / 44.6 / 46.3 / 48.8;
//   24 of 64, 1536: 850 21.8 / 23.3 / 23.8 / 24.3 -> 22.5 / 22.6 / 23.7 / 24.3, 1000 22.0 / 23.5 / 24.3 / 24.7 -> 22.7 / 22.9 / 24.0 / 24.6, 4000 26.7 / 28.6 / 30.9 / 37.4 -> 27.0 / 27.2 / 28.7 / 29.6;
//   32 of 80, 2560: 850 37.0 / 37.0 / 39.2 / 40.4 -> 36.4 / 36.7 / 37.8 / 39.9, 1000 37.5 / 37.4 / 39.6 / 40.8 -> 36.4 / 36.8 / 38.1 / 40.2, 4000 43.0 / 48.1 / 55.0 / 55.6 -> 42.9 / 43.2 / 44.7 / 46.9;
//   32 of 128, 4096: 850 72.0 / 72.0 / 74.7 / 77.1 -> 71.7 / 72.3 / 73.9 / 77.0, 1000 72.2 / 72.4 / 75.8 / 77.9 -> 72.8 / 73.2 / 74.7 / 77.6, 4000 80.2 / 87.5 / 103.3 / 104.9 -> 81.1 / 81.9 / 83.5 / 86.4.
// Over 19 shapes, two to eight tokens and positions from 1000 to 4000 (16 .. 21 heads, 118 of them): the slower one by 0.5 % in the mean, 1.0 % with the
// line at 896 positions alone; what it takes loses 2 % at most (before 7 %), what it leaves 3 % but for 18 heads of 64 (up to 12 % with 4 tokens behind 2000).  From
// 22 heads on: 3 % for 2 tokens behind 1000 at 24 heads, 5 % for 5 at 24 heads of 80, else below 2 %.  Eight heads of 128 dimensions are too few
// workgroups with too much to read (hidden 1024 behind 1000 / 4000: 3 tokens 7.5 / 9.4 % more, 8 8.4 / 0.9 % more): left with the other kernel, as are
// eight of 80 (2 tokens behind 1000 6 % less, but 8 3 % more behind 1200).
bool group_attention_takes(const Dims &dm, int nb, int first)
{
    return nb >= 2 && first >= 28 * kGaRow && (dm.H < 16 ? dm.d == 64 : dm.H >= 22 || dm.H * nb * first >= 160000);
}

constexpr float kGaWeight = 16384.f;   // a weight's factor
// Both columns of a query, eight lanes apart, work its values out alike.  One of them feeds the head of v (below 2^15 in size), the other what it
// leaves: (float)head * -b + v * a is v itself, or 2^11 (v - head), exactly.  Their sums join to the same value in both.
struct GaSide {
    float a, b, own, other;
    __device__ __forceinline__ explicit GaSide(bool heads) : a(heads ? 1.f : 2048.f), b(heads ? 0.f : -2048.f), own(heads ? 1.f : 1.f / 2048.f), other(heads ? 1.f / 2048.f : 1.f) {}
    __device__ __forceinline__ _Float16 part(float v) const { return (_Float16)fmaf((float)(_Float16)v, b, v * a); }
    __device__ __forceinline__ float joined(float sum) const { return fmaf(sum, own, dpp_mov<kDppRor8>(sum) * other); }
};

struct GaParams {
    int nb, first, pieces;  // tokens; the first one's position; pieces of the positions ahead of it
    const __half *kv;
};

template <int D>
constexpr int ga_lds()                 // V; then the wavefronts' sums
{
    const int v = kGaWaves * D * kGaStride * 2, w = kGaWaves * kBatMax * (D + 2) * 4;
    return v > w ? v : w;
}

// what a wavefront holds of a row of positions
template <int D>
struct GaRow {
    static constexpr int KS = (D + 31) / 32, UN = (D / 8 * (kGaRow / 2) + 63) / 64;
    u32x4 k[2][KS], v[UN][2];
    // Positions past the last one ahead of the group read that one again.
    __device__ __forceinline__ void request(const __half *Kh, const __half *Vh, unsigned slab, int row, int last, int lane)
    {
        const int n = lane & 15, kg = lane >> 4;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KS; ++s)
                k[t][s] = load16(Kh + (unsigned)min(2 * s + (kg >> 1), D / 16 - 1) * slab + (unsigned)min(row * kGaRow + 16 * t + n, last) * 16u + (kg & 1) * 8u);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int e = min(lane + 64 * u, D / 8 * (kGaRow / 2) - 1), pc = e / (kGaRow / 2), t = row * kGaRow + 2 * (e % (kGaRow / 2));
#pragma unroll
            for (int i = 0; i < 2; ++i) v[u][i] = load16(Vh + (unsigned)(pc >> 1) * slab + (unsigned)min(t + i, last) * 16u + (pc & 1) * 8u);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // V, transposed, to LDS: [dimension][kGaStride]; positions past the last one as zeros
    __device__ __forceinline__ void store(__half *vt, int row, int last, int lane)
    {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int e = lane + 64 * u, pc = e / (kGaRow / 2), tp = e % (kGaRow / 2), t = row * kGaRow + 2 * tp;
            if (D / 8 * (kGaRow / 2) % 64 != 0 && e >= D / 8 * (kGaRow / 2)) break;
            const u32x4 a = t <= last ? v[u][0] : u32x4{0u, 0u, 0u, 0u}, b = t + 1 <= last ? v[u][1] : u32x4{0u, 0u, 0u, 0u};
            unsigned *to = reinterpret_cast<unsigned *>(vt + 8 * pc * kGaStride) + tp;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                to[2 * j * (kGaStride / 2)] = __builtin_amdgcn_perm(b[j], a[j], 0x05040100u);
                to[(2 * j + 1) * (kGaStride / 2)] = __builtin_amdgcn_perm(b[j], a[j], 0x07060302u);
            }
        }
    }
};

// largest and sum over the four lanes that share lane % 16
__device__ __forceinline__ float ga_max4(float v)
{
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float ga_sum4(float v)
{
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// One wavefront, one query: its sums over the wavefront's rows in fp32, position by position
template <int D>
__device__ __forceinline__ void ga_alone(const float *q, const __half *Kh, const __half *Vh, unsigned slab, int row0, int hi, int last, int lane,
                                         float *o_out, float *m_out, float *l_out)
{
    constexpr int NE = (D + 63) / 64;
    const float scale = 1.44269504088896340736f / sqrtf((float)D);
    float qs[NE], o[NE], m = kAttnLowest, l = 0.f;
    unsigned at[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int dim = min(lane + 64 * e, D - 1);
        at[e] = (unsigned)(dim >> 4) * slab + (dim & 15);
        qs[e] = lane + 64 * e < D ? q[dim] * scale : 0.f;
        o[e] = 0.f;
    }
    for (int row = row0; row < hi; row += kGaWaves) {
        for (int t = row * kGaRow; t <= min(row * kGaRow + kGaRow - 1, last); ++t) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < NE; ++e) s = lane + 64 * e < D ? fmaf(qs[e], __half2float(Kh[at[e] + (unsigned)t * 16u]), s) : s;
            s = wave_sum(s);
            const float mn = fmaxf(m, s), corr = __builtin_amdgcn_exp2f(m - mn), p = __builtin_amdgcn_exp2f(s - mn);
            m = mn;
            l = l * corr + p;
#pragma unroll
            for (int e = 0; e < NE; ++e) o[e] = fmaf(p, __half2float(Vh[at[e] + (unsigned)t * 16u]), o[e] * corr);
        }
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if (lane + 64 * e < D) o_out[lane + 64 * e] = o[e];
    if (lane == 0) { *m_out = m; *l_out = l; }
}

// (80 dimensions in 128 registers, which is enough: with the 160 that the compiler takes otherwise eight tokens of hidden 2560 behind 1000 are
// 489 us of twelve layers, with 128 485)
template <int D>
__global__ void __launch_bounds__(kAttnBatchThreads, D == 80 ? 4 : 3) k_attention_group(StepParams P, GaParams G, DownPlan down)
{
    extern __shared__ __align__(16) char ga_mem[];
    if ((int)blockIdx.x >= down.first) {
        mlp_down<false>(P, down, (int)blockIdx.x - down.first, G.nb, ga_mem);
        return;
    }
    constexpr int W = kGaWaves, KS = GaRow<D>::KS, NT = D / 16, Q8 = kBatMax;
    static_assert(ga_lds<D>() <= down_lds<false>() - 1024, "");
    const Dims &dm = P.dm;
    const int H = dm.H, nb = G.nb, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int piece = (int)blockIdx.x / H, head = (int)blockIdx.x - piece * H, pieces = G.pieces;
    const __half *Kh = G.kv + kv_offset(dm, 0, P.b, head, 0, 0), *Vh = G.kv + kv_offset(dm, 1, P.b, head, 0, 0);
    const unsigned slab = (unsigned)dm.max_seq * 16u;
    const float *q = P.q + head * D;
    float *part = P.part + (size_t)head * P.part_slots * (D + 2);          // of token i: i H part_slots (D + 2) further
    const size_t part_step = (size_t)H * P.part_slots * (D + 2);
    int *last_one = reinterpret_cast<int *>(ga_mem + down_lds<false>() - 1024);
    const float scale = 1.44269504088896340736f / sqrtf((float)D);
    auto deliver = [&](int i, int dim, float v) {          // as the output projection takes them: heads and remainders
        __half hi, lo;
        split_half(v, hi, lo);
        __half *out = reinterpret_cast<__half *>(P.o) + ng_at(i, head * D + dim, dm.h, nb);
        out[0] = hi; out[8 * nb] = lo;
    };
    if (piece == pieces) {                                 // the group's own rows
        float *sp = reinterpret_cast<float *>(ga_mem), *sm = sp + Q8 * Q8, *sl = sm + Q8;
        u32x4 v[Q8];
        const int i = min(tid / (D / 8), nb - 1), pc = tid % (D / 8);      // this thread's query and eight dimensions
        const bool mine = tid < nb * (D / 8);
#pragma unroll
        for (int j = 0; j < Q8; ++j) v[j] = load16(Vh + (unsigned)(pc >> 1) * slab + (unsigned)(G.first + min(j, i)) * 16u + (pc & 1) * 8u);
        if (wave == 0) {                                   // scores: query lane / 8, row lane % 8
            const int si = lane >> 3, sj = lane & 7;
            const __half *kr = Kh + (unsigned)(G.first + min(sj, nb - 1)) * 16u;
            const float *qr = q + (size_t)min(si, nb - 1) * dm.h;
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < D / 8; ++c)
                s += dot8(load16(kr + (unsigned)(c >> 1) * slab + (c & 1) * 8u), *reinterpret_cast<const float4 *>(qr + 8 * c),
                          *reinterpret_cast<const float4 *>(qr + 8 * c + 4), 0.f);
            s = sj <= si ? s * scale : -INFINITY;
            float m = fmaxf(fmaxf(s, kAttnLowest), dpp_mov<kDppXor1>(s));
            m = fmaxf(m, dpp_mov<kDppXor2>(m));
            m = fmaxf(m, dpp_mov<kDppHalfMirror>(m));
            const float p = __builtin_amdgcn_exp2f(s - m);
            float l = p + dpp_mov<kDppXor1>(p);
            l += dpp_mov<kDppXor2>(l);
            l += dpp_mov<kDppHalfMirror>(l);
            sp[lane] = p;
            if (sj == 0) { sm[si] = m; sl[si] = l; }
        }
        __syncthreads();
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
        for (int j = 0; j < Q8; ++j) {
            const float p = sp[i * Q8 + j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 x = unpack_h2(v[j][e]);
                if (j <= i) { o[2 * e] = fmaf(p, x.x, o[2 * e]); o[2 * e + 1] = fmaf(p, x.y, o[2 * e + 1]); }
            }
        }
        if (mine) {
            float *slot = part + i * part_step + (size_t)piece * (D + 2);
#pragma unroll
            for (int e = 0; e < 8; ++e) xwg_store(slot + 8 * pc + e, o[e]);
            if (pc == 0) { xwg_store(slot + D, sm[i]); xwg_store(slot + D + 1, sl[i]); }
        }
    } else {
        const int R = (G.first + kGaRow - 1) / kGaRow, lo = R * piece / pieces, hi = R * (piece + 1) / pieces, last = G.first - 1;
        const int col = lane & 15, kg = lane >> 4;
        GaRow<D> r;                                        // (one row ahead: pieces are cut so that a wavefront has few)
        r.request(Kh, Vh, slab, lo + wave, last, lane);
        const GaSide side(col < 8);
        // Q^T: dimensions 32 s + 8 kg .. + 7 of query col % 8
        ga_f16x8 Q[KS];
        float qscale;
        {
            float x[KS][8], most = 0.f;
            const float *qr = q + (size_t)min(col & 7, nb - 1) * dm.h;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bool real = D % 32 == 0 || 32 * s + 8 * kg < D;
                const f32x4 *at = reinterpret_cast<const f32x4 *>(qr + (real ? 32 * s + 8 * kg : 0));
                const f32x4 x0 = *as_global(at), x1 = *as_global(at + 1);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    x[s][e] = real ? (e < 4 ? x0[e & 3] : x1[e & 3]) : 0.f;
                    most = fmaxf(most, fabsf(x[s][e]));
                }
            }
            most = ga_max4(most);
            const int ex = (most > 0.f && most < INFINITY ? __builtin_amdgcn_frexp_expf(most) : 0) - 15;
            qscale = __builtin_amdgcn_ldexpf(scale, ex);
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) Q[s][e] = side.part(split_value(__builtin_amdgcn_ldexpf(x[s][e], -ex)));
        }
        f32x4 O[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) O[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m_run = kAttnLowest, l_run = 0.f;            // l_run: of this lane's positions
        __half *vt = reinterpret_cast<__half *>(ga_mem) + wave * D * kGaStride;
        for (int row = lo + wave; row < hi; row += W) {
            r.store(vt, row, last, lane);
            asm volatile("" ::: "memory");                 // (LDS takes a wavefront's accesses in order)
            f32x4 S[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x4 half[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};          // (128 dimensions in two sums: smaller roundings)
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    u32x4 k = r.k[t][s];
                    if (D % 32 != 0 && s == KS - 1 && 32 * s + 8 * kg >= D) k = u32x4{0u, 0u, 0u, 0u};
                    half[KS > 3 ? s / 2 : 0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(ga_f16x8, k), Q[s], half[KS > 3 ? s / 2 : 0], 0, 0, 0);
                }
                if (KS > 3) __builtin_amdgcn_sched_barrier(0);             // (a tile at a time: registers)
                S[t] = KS > 3 ? half[0] + half[1] : half[0];
            }
            r.request(Kh, Vh, slab, row + W, last, lane);
            float most = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float s = side.joined(S[t][j]) * qscale;
                    S[t][j] = row * kGaRow + 16 * t + 4 * kg + j <= last ? s : -INFINITY;
                    most = fmaxf(most, S[t][j]);
                }
            const float mn = fmaxf(m_run, ga_max4(most)), corr = __builtin_amdgcn_exp2f(m_run - mn);
            ga_f16x8 p;
            float sum = 0.f;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = split_value(__builtin_amdgcn_exp2f(S[t][j] - mn));
                    sum += v;
                    p[4 * t + j] = side.part(v * kGaWeight);
                }
            l_run = l_run * corr + sum;
            m_run = mn;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const __half *at = vt + (16 * t + col) * kGaStride + 4 * kg;
                const ga_f16x4 v0 = *reinterpret_cast<const ga_f16x4 *>(at), v1 = *reinterpret_cast<const ga_f16x4 *>(at + 16);
                const ga_f16x8 v = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                O[t] *= corr;
                O[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v, p, O[t], 0, 0, 0);
            }
            asm volatile("" ::: "memory");
        }
        // wavefronts: maxima and weights [wave][query], then [wave][query][D] in the place of V
        float *wp = reinterpret_cast<float *>(ga_mem), *wm = wp + W * Q8 * D, *wl = wm + W * Q8;
        const float l = ga_sum4(l_run);
        bool finite = true;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                O[t][j] = side.joined(O[t][j]) * (1.f / kGaWeight);
                finite = finite && fabsf(O[t][j]) < INFINITY;
            }
        const unsigned long long again = __ballot(!finite);            // (bit l: query l % 8)
        __syncthreads();                                   // V has been read
        if (col < 8) {
#pragma unroll
            for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4 *>(wp + (wave * Q8 + col) * D + 16 * t + 4 * kg) = O[t];
            if (kg == 0) { wm[wave * Q8 + col] = m_run; wl[wave * Q8 + col] = l; }
        }
        if (again) {                                       // (uniform)
            asm volatile("" ::: "memory");
            for (int i = 0; i < nb; ++i)
                if (again & (0x0101010101010101ull << i))
                    ga_alone<D>(q + (size_t)i * dm.h, Kh, Vh, slab, lo + wave, hi, last, lane, wp + (wave * Q8 + i) * D, wm + wave * Q8 + i, wl + wave * Q8 + i);
        }
        __syncthreads();
        for (int e = tid; e < nb * D; e += kAttnBatchThreads) {
            const int i = e / D, dim = e - i * D;
            float M = wm[i], L = 0.f, s = 0.f;
#pragma unroll
            for (int w = 1; w < W; ++w) M = fmaxf(M, wm[w * Q8 + i]);
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float ew = __builtin_amdgcn_exp2f(wm[w * Q8 + i] - M);
                L += wl[w * Q8 + i] * ew;
                s += wp[(w * Q8 + i) * D + dim] * ew;
            }
            float *slot = part + i * part_step + (size_t)piece * (D + 2);
            xwg_store(slot + dim, s);
            if (dim == 0) { xwg_store(slot + D, M); xwg_store(slot + D + 1, L); }
        }
    }
    // the head's last workgroup adds the pieces in order
    xwg_wait_stores();
    __syncthreads();
    if (tid == 0) *last_one = __hip_atomic_fetch_add(&P.seg_cnt[head], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)pieces;
    __syncthreads();
    if (!*last_one) return;
    for (int e = tid; e < nb * D; e += kAttnBatchThreads) {
        const int i = e / D, dim = e - i * D;
        const float *first = part + i * part_step;
        float M = kAttnLowest, L = 0.f, s = 0.f;
        constexpr int CB = kGaPieces + 1;                  // all of them in flight together
        float mj[CB], lj[CB], oj[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const float *sj = first + (size_t)min(j, pieces) * (D + 2);
            mj[j] = xwg_load(sj + D);
            lj[j] = xwg_load(sj + D + 1);
            oj[j] = xwg_load(sj + dim);
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            if (j <= pieces) {
                const float mn = fmaxf(M, mj[j]);
                const float c0 = __builtin_amdgcn_exp2f(M - mn), c1 = __builtin_amdgcn_exp2f(mj[j] - mn);
                L = L * c0 + lj[j] * c1;
                s = s * c0 + oj[j] * c1;
                M = mn;
            }
        }
        deliver(i, dim, s / L);
    }
    if (tid == 0) __hip_atomic_store(&P.seg_cnt[head], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

AttnPlan plan_attention_group(const Dims &dm, int, int first)
{
    AttnPlan A;
    A.pieces = ga_pieces(first, dm.H);
    A.attn = dm.H * (A.pieces + 1);
    A.downs = down_parts_beside(dm.h, dm.f, false, A.attn, first);
    return A;
}

hipError_t launch_attention_group(const StepParams &P, int nb, int first, const __half *w, const __half *kv, int *downs, hipStream_t s)
{
    if (nb < 2 || nb > kBatMax || first < 0 || first + nb > P.dm.max_seq || P.part_slots < kGaPieces + 1 + kDownParts) return hipErrorInvalidValue;
    const AttnPlan plan = plan_attention_group(P.dm, nb, first);
    GaParams G;
    G.nb = nb; G.first = first; G.kv = kv;
    G.pieces = plan.pieces;
    DownPlan down;
    down.w = w;
    down.first = plan.attn;
    down.parts = plan.downs;
    *downs = down.parts;
    const dim3 grid(down.first + P.dm.h / kDownRows * down.parts), block(kAttnBatchThreads);
    switch (P.dm.d) {
    case 64: hipLaunchKernelGGL(k_attention_group<64>, grid, block, down_lds<false>(), s, P, G, down); break;
    case 80: hipLaunchKernelGGL(k_attention_group<80>, grid, block, down_lds<false>(), s, P, G, down); break;
    case 128: hipLaunchKernelGGL(k_attention_group<128>, grid, block, down_lds<false>(), s, P, G, down); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cfpp
