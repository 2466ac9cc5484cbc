// The stream of a product for few tokens: weights from memory through LDS rings into matrix instructions (narrow_gemm.hip,
// prefill_narrow.hip; MLP-down of both: mlp_down.h, prefill_beside.hip).
//
// A workgroup (up to 8 wavefronts, one workgroup to a CU) owns a contiguous range of rows of one matrix and its wavefronts
// split K: a wavefront streams its columns of all rows, 64 columns (a chunk: whole 128-byte lines) at a time, through an LDS
// ring of its own that is filled by memory-to-LDS loads.  No wavefront waits for another before the sums are added, no
// register holds what is in flight, and a row counts for nothing but its own bytes, whatever their number.  Measured with
// loads alone (one launch, launch included): 92 MB of 17920 x 2560: 15.7 us, 235 MB of 28672 x 4096: 36 us = 6.5 TB/s; every
// set of 8 tokens adds 0.9 us to the first (all its activations, read by every CU from the L2; 1.6 where a block of them is
// eight pieces of 64 bytes instead of one KiB, hence ng_at).
//
// v_mfma_f32_16x16x32_f16: A = 16 rows x 32 columns of weights, from the ring; B = the same 32 columns of 8 tokens, the
// fp16 heads of their fp32 activations in columns 0..7 and the remainders in 8..15 (half_split.h): one
// instruction per KiB of weights and set.  The two columns of a token and the wavefronts' parts of K are added in a fixed
// order at the end: one bit pattern per build.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "device_utils.h"
#include "half_split.h"
#include "lds_dma.h"
#include "narrow_params.h"

namespace cfpp {

typedef _Float16 ng_f16x8 __attribute__((ext_vector_type(8)));

constexpr int kNgChunk = 64, kNgTileMax = 8;   // columns of a chunk; most tiles of 16 rows to a workgroup
// what the activations are in memory: planes (ng_at), or the layer input itself (fp32 or fp16), which the
// wavefronts multiply by gamma and split on the way
enum { kNgPlanes, kNgRaw32, kNgRaw16 };

// the sums of a tile and set in LDS: 8 tokens of 16 rows, 20 floats apart
constexpr int kNgTileFloats = 160;

// chunks [c0, c0 + n) of a workgroup's rows of one matrix, and where their activations are
struct NgPiece {
    const void *w, *b;      // first row; activations
    unsigned row_bytes, b_bytes, set_bytes;    // set_bytes: planes, between the sets of 8 tokens
    int c0, n;
};

template <int N>
__device__ __forceinline__ void ng_wait() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
template <int MOST>
__device__ __forceinline__ void ng_wait_for(int left)      // left <= MOST: a constant where this is expanded
{
    if (left == MOST) ng_wait<MOST>();
    else if constexpr (MOST > 0) ng_wait_for<MOST - 1>(left);
}
__device__ __forceinline__ void ng_lds_read() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The stream of one wavefront.  A stage is CH chunks; of each, NB loads bring the activations of S sets of 8 tokens and 2 T
// the weights of T tiles of 16 rows (a load: 8 rows x 128 bytes).  Every load of a stage has its place in the ring, and is requested
// again - for the next stage - as soon as what it brought has been read: NI - 2 or NI - NB loads are always in
// flight behind the one that is waited for, by count.  Loads without a purpose (rows past the last, chunks past
// the end) read one line over and over.
template <int T, int S, int SRC, int CH>
struct NgStream {
    static constexpr int NB = SRC == kNgRaw16 ? 1 : 2 * S, PER = NB + 2 * T, NI = CH * PER, kStage = NI * 1024;
    static_assert(NI <= 62, "the memory counter's range");
    static_assert(S == 1 || SRC == kNgPlanes, "");
    static constexpr int kSetFloats = T * kNgTileFloats;   // sums of a set
    NgPiece p0, p1;
    unsigned ring;          // LDS address of this wavefront's ring
    const char *mem;        // the same as a pointer
    const char *gamma;      // this wavefront's columns of gamma in LDS (layer input only)
    int lane, octets, tail; // whole 8-row groups, rows beyond them
    unsigned v_b, place, a_at;
    f32x4 acc[T][S];
    float mean, m2;         // of the layer input's columns this lane has seen

    __device__ __forceinline__ void issue_b(int i, int ch) const
    {
        const bool second = i >= p0.n, live = i < p0.n + p1.n;
        const int c = second ? p1.c0 + i - p0.n : p0.c0 + i;
        const i32x4 rs = dma_rsrc(second ? p1.b : p0.b, second ? p1.b_bytes : p0.b_bytes);
        const unsigned step = SRC == kNgPlanes ? b_block : 128u, set = second ? p1.set_bytes : p0.set_bytes;
        constexpr int KB = SRC == kNgRaw16 ? 1 : 2;        // loads of a set
#pragma unroll
        for (int k = 0; k < NB; ++k)
            lds_dma16(rs, ring + (unsigned)(ch * PER + k) * 1024u, live ? v_b : 0u,
                      live ? (unsigned)(KB * c + k % KB) * step + (S > 1 ? (unsigned)(k / KB) * set : 0u) : 0u);
    }
    unsigned b_block;       // planes: bytes of a block of 32 columns

    __device__ __forceinline__ void issue_w(int i, int ch, int t) const
    {
        const bool second = i >= p0.n, live = i < p0.n + p1.n;
        const int c = second ? p1.c0 + i - p0.n : p0.c0 + i;
        const unsigned row_bytes = second ? p1.row_bytes : p0.row_bytes;
        const i32x4 rs = dma_rsrc(second ? p1.w : p0.w, row_bytes * (unsigned)(8 * octets + tail));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int o = 2 * t + k;                       // row group; its last rows may not be there
            const unsigned r = o < octets ? (unsigned)(lane >> 3) : (unsigned)min(lane >> 3, tail - 1);
            const bool real = live && (o < octets || (o == octets && tail > 0));
            const unsigned v = r * row_bytes + (place ^ (unsigned)(16 * k));
            lds_dma16_once(rs, ring + (unsigned)(ch * PER + NB + o) * 1024u, real ? v : 0u, real ? (unsigned)(8 * o) * row_bytes + (unsigned)c * 128u : 0u);
        }
    }

    // nt: tokens of a block of planes; n: tokens there are
    __device__ __forceinline__ void begin(int rows, int n, int nt, unsigned x_stride, int tid)
    {
        lane = tid & 63;
        octets = rows >> 3; tail = rows & 7;
        // row r of a row group keeps its 16-byte pieces at (piece ^ r ^ (group & 1)): 16 rows' reads of one piece hit all banks
        place = (unsigned)(((lane & 7) ^ (lane >> 3)) * 16);
        const int row = lane & 15, kg = lane >> 4;
        a_at = (unsigned)(NB * 1024 + (row >> 3) * 1024 + (row & 7) * 128 + ((kg ^ (row & 7) ^ (row >> 3)) & 7) * 16);
        b_block = (unsigned)nt * 128u;
        if (SRC == kNgPlanes) v_b = (unsigned)((2 * kg + ((lane >> 3) & 1)) * nt + min(lane & 7, nt - 1)) * 16u;
        else v_b = (unsigned)min(lane >> 3, n - 1) * x_stride + place;     // 128 bytes of every token
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int e = 0; e < S; ++e) acc[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        mean = m2 = 0.f;
        if (p0.n + p1.n > 0) {
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) {
                issue_b(ch, ch);
#pragma unroll
                for (int t = 0; t < T; ++t) issue_w(ch, ch, t);
            }
        }
    }

    // this lane's operand: column lane % 16 (head or remainder of token lane % 8), 8 columns of K at 8 (lane / 16), of both
    // halves of chunk i; of the layer input also its contribution to mean and variance
    __device__ __forceinline__ void activations(int i, int ch, ng_f16x8 (&b)[2 * S])
    {
        const char *at = mem + ch * PER * 1024;
        if (SRC == kNgPlanes) {
#pragma unroll
            for (int k = 0; k < 2 * S; ++k) b[k] = *reinterpret_cast<const ng_f16x8 *>(at + k * 1024 + lane * 16);
            return;
        }
        const int token = lane & 7, kg = lane >> 4;
        float x[16];
        if (SRC == kNgRaw16) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(at + (token * 8 + ((4 * k + kg) ^ token)) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float2 f = unpack_h2(v[e]);
                    x[8 * k + 2 * e] = f.x; x[8 * k + 2 * e + 1] = f.y;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(at + k * 1024 + (token * 8 + ((2 * kg + p) ^ token)) * 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[8 * k + 4 * p + e] = v[e];
                }
        }
        u32x4 g[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) g[k] = *reinterpret_cast<const u32x4 *>(gamma + (8 * i + 4 * k + kg) * 16);
        ng_lds_read();                                     // the place in the ring is free
        const bool rest = lane & 8;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float2 gg = unpack_h2(g[j >> 3][(j & 7) >> 1]);
            const float v = split_value(x[j] * (j & 1 ? gg.y : gg.x));
            const _Float16 hi = (_Float16)v, lo = (_Float16)(v - (float)hi);
            b[j >> 3][j & 7] = rest ? lo : hi;
        }
        // mean and sum of squared deviations of these 16, joined to those of the 16 i before
        float s = 0.f, q = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) s += x[j];
        const float mc = s * 0.0625f;
#pragma unroll
        for (int j = 0; j < 16; ++j) q = fmaf(x[j] - mc, x[j] - mc, q);
        const float w = 1.f / (float)(i + 1), dl = mc - mean;
        mean = fmaf(dl, w, mean);
        m2 += fmaf(dl * dl, 16.f * (float)i * w, q);
    }

    template <bool LAST>
    __device__ __forceinline__ void stage(int i)
    {
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            const bool live = CH == 1 || i + ch < p0.n + p1.n;             // (uniform)
            ng_f16x8 b[2 * S];
            if (LAST) ng_wait_for<NI>(NI - ch * PER - NB);
            else ng_wait<NI - NB>();
            if (live) activations(i + ch, ch, b);
            ng_lds_read();
            if (!LAST) issue_b(i + CH + ch, ch);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (LAST) ng_wait_for<NI>(NI - ch * PER - NB - 2 * (t + 1));
                else ng_wait<NI - 2>();
                const char *at = mem + (ch * PER + 2 * t) * 1024;
                const ng_f16x8 w0 = *reinterpret_cast<const ng_f16x8 *>(at + a_at), w1 = *reinterpret_cast<const ng_f16x8 *>(at + (a_at ^ 64u));
                ng_lds_read();
                if (!LAST) issue_w(i + CH + ch, ch, t);
                if (live) {
#pragma unroll
                    for (int e = 0; e < S; ++e) acc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w0, b[2 * e], acc[t][e], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < S; ++e) acc[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1, b[2 * e + 1], acc[t][e], 0, 0, 0);
                }
            }
        }
    }
    __device__ __forceinline__ void run()
    {
        const int n = p0.n + p1.n;
        if (n == 0) return;
        int i = 0;
        for (; i + CH < n; i += CH) stage<false>(i);
        stage<true>(i);
    }

    // The sums of sets [s0, s0 + N) of the wavefront's tiles, [set][tile][token][20]: rows side by side.  A token's heads and
    // remainders are eight lanes apart: added here, so that half as much goes through LDS.
    template <int N>
    __device__ __forceinline__ void leave(float *red, int wave, int s0) const
    {
        const int col = lane & 15, r4 = 4 * (lane >> 4);
#pragma unroll
        for (int e = 0; e < S; ++e) {
            if (e < s0 || e >= s0 + N) continue;           // (s0: a constant where this is expanded)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                f32x4 v = acc[t][e];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] += dpp_mov<kDppRor8>(v[j]);
                if (col < kNgSet) *reinterpret_cast<f32x4 *>(red + (wave * N + e - s0) * kSetFloats + (t * kNgSet + col) * 20 + r4) = v;
            }
        }
    }
};

// Row `row` of the workgroup for token b of a set: the W wavefronts' sums, in order.  red: the set's sums of the first
// wavefront, `stride` floats ahead of the next one's.
template <int W>
__device__ __forceinline__ float ng_total(const float *red, int stride, int row, int b)
{
    const float *p = red + ((row >> 4) * kNgSet + b) * 20 + (row & 15);
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) s += p[w * stride];
    return s;
}
template <int W>
__device__ __forceinline__ float2 ng_total2(const float *red, int stride, int row, int b)         // rows row, row + 1 (row even)
{
    const float *p = red + ((row >> 4) * kNgSet + b) * 20 + (row & 15);
    float2 s{0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const float2 v = *reinterpret_cast<const float2 *>(p + w * stride);
        s.x += v.x; s.y += v.y;
    }
    return s;
}

// MLP-down's parts of a row of a token, requested together (past the last: the last again), and their sum in order
__device__ __forceinline__ void down_parts(const NarrowParams &P, int token, int row, float (&v)[kDownParts])
{
    const float *at = P.part + down_at(token, row, 0, P.dm.H, P.dm.d, P.part_slots);
#pragma unroll
    for (int z = 0; z < kDownParts; ++z) v[z] = at[min(z, P.downs - 1) * (P.dm.d + 2)];
}
__device__ __forceinline__ float down_sum(const NarrowParams &P, const float (&v)[kDownParts])
{
    float s = v[0];
#pragma unroll
    for (int z = 1; z < kDownParts; ++z) s += z < P.downs ? v[z] : 0.f;
    return s;
}

// Rows of a workgroup such that the workgroups of both matrices of the first product come to at most `grid`; even: a rotary
// pair stays in one workgroup.  0 where that would be more than kNgTileMax tiles of 16.
inline int ng_in_rows(const Dims &dm, int grid, int *wgs_q, int *wgs)
{
    for (int rows = 2; rows <= 16 * kNgTileMax; rows += 2) {
        const int q = (3 * dm.h + rows - 1) / rows, u = (dm.f + rows - 1) / rows;
        if (q + u <= grid) { *wgs_q = q; *wgs = q + u; return rows; }
    }
    return 0;
}

}  // namespace cfpp
