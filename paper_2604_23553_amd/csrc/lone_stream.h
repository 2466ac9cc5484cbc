// The stream of a product for one token: weights from memory through LDS rings into fused multiply-adds with fp32
// activations (lone_gemm.hip, narrow_attention.hip).
#pragma once
#include "narrow_stream.h"

namespace cfpp {

// The stream of one wavefront: chunks of 64 columns of T pairs of 8 rows, CH chunks to a stage, through an LDS ring of its own.  A
// load brings 8 rows x 128 bytes, and a lane reads back the 16 bytes that it asked for.  ACT: every fourth chunk is
// preceded by a load of the four chunks' activations (256 fp32 values); else they are in LDS, at y.  Every load has its
// place in the ring and is requested again, for the next stage, as soon as what it brought has been read: NI - 2 loads (behind
// activations NI - 1) are always in flight behind those that are waited for, by count.  Loads without a purpose
// (rows past the last, chunks past the end) read one line over and over.  A wavefront with no more chunks than a stage
// requests just these and waits for all of them at once.
template <int T, int CH, bool ACT>
struct LoneStream {
    static constexpr int PER = 2 * T, NI = CH * PER + (ACT ? CH / 4 : 0), kStage = NI * 1024;
    static_assert(NI <= 62, "the memory counter's range");
    static_assert(!ACT || CH % 4 == 0, "");
    NgPiece p0;
    const void *act;        // ACT: the activations, from the matrix's first column on
    unsigned act_bytes;     // their size
    unsigned ring;          // LDS address of this wavefront's ring
    const char *mem;        // the same as a pointer
    const float *y;         // !ACT: this wavefront's activations
    int lane, octets, tail; // whole 8-row groups, rows beyond them
    float acc[2 * T];       // this lane's columns of row lane / 8 of each group

    static constexpr unsigned place_w(int ch, int o) { return (unsigned)((ACT ? ch / 4 + 1 : 0) + ch * PER + o) * 1024u; }
    static constexpr unsigned place_a(int quad) { return (unsigned)(quad * (1 + 4 * PER)) * 1024u; }

    __device__ __forceinline__ void issue_a(int i, int quad) const
    {
        const int k = i + (lane >> 4);
        const unsigned v = (unsigned)(p0.c0 + k) * 256u + (unsigned)(lane & 15) * 16u;
        lds_dma16(dma_rsrc(act, act_bytes), ring + place_a(quad), k < p0.n ? v : 0u, 0u);
    }
    __device__ __forceinline__ void issue_w(int i, int ch, int t) const
    {
        const bool live = i < p0.n;
        const int c = p0.c0 + i;
        const unsigned row_bytes = p0.row_bytes;
        const i32x4 rs = dma_rsrc(p0.w, row_bytes * (unsigned)(8 * octets + tail));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int o = 2 * t + k;                       // row group; its last rows may not be there
            const unsigned r = o < octets ? (unsigned)(lane >> 3) : (unsigned)min(lane >> 3, tail - 1);
            const bool real = live && (o < octets || (o == octets && tail > 0));
            lds_dma16_once(rs, ring + place_w(ch, o), real ? r * row_bytes + (unsigned)(lane & 7) * 16u : 0u,
                           real ? (unsigned)(8 * o) * row_bytes + (unsigned)c * 128u : 0u);
        }
    }
    __device__ __forceinline__ void begin(int rows, int tid)
    {
        lane = tid & 63;
        octets = rows >> 3; tail = rows & 7;
#pragma unroll
        for (int o = 0; o < 2 * T; ++o) acc[o] = 0.f;
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            if (ch >= p0.n) break;                         // (uniform)
            if (ACT && ch % 4 == 0) issue_a(ch, ch / 4);
#pragma unroll
            for (int t = 0; t < T; ++t) issue_w(ch, ch, t);
        }
    }
    // what was requested ahead of begin() is there (!ACT: begin() requested whole chunks, CH or as many as there are)
    template <int N = CH>
    __device__ __forceinline__ void wait_ahead() const
    {
        if (p0.n >= N) ng_wait<N * PER>();
        else if constexpr (N > 0) wait_ahead<N - 1>();
    }
    enum { kSteady, kLast, kOnly };
    template <int KIND>
    __device__ __forceinline__ void stage(int i)
    {
        constexpr bool LAST = KIND != kSteady;
        float4 a[ACT ? 8 : 2];
        if (KIND == kOnly) ng_wait<0>();
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            const bool live = CH == 1 || i + ch < p0.n;    // (uniform)
            if (KIND == kOnly && !live) break;
            if (ACT && ch % 4 == 0) {
                if (KIND == kLast) ng_wait_for<NI>(NI - ch * PER - ch / 4 - 1);
                else if (KIND == kSteady) ng_wait<NI - 1>();
                const float4 *at = reinterpret_cast<const float4 *>(mem + place_a(ch / 4) + (lane & 7) * 32);
#pragma unroll
                for (int k = 0; k < 4; ++k) { a[2 * k] = at[16 * k]; a[2 * k + 1] = at[16 * k + 1]; }
                ng_lds_read();                             // the place in the ring is free
                if (!LAST) issue_a(i + CH + ch, ch / 4);
            } else if (!ACT && live) {
                const float4 *at = reinterpret_cast<const float4 *>(y + (i + ch) * kNgChunk + (lane & 7) * 8);
                a[0] = at[0]; a[1] = at[1];
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (KIND == kLast) ng_wait_for<NI>(NI - ch * PER - (ACT ? ch / 4 + 1 : 0) - 2 * (t + 1));
                else if (KIND == kSteady) ng_wait<NI - 2>();
                const u32x4 w0 = *reinterpret_cast<const u32x4 *>(mem + place_w(ch, 2 * t) + lane * 16);
                const u32x4 w1 = *reinterpret_cast<const u32x4 *>(mem + place_w(ch, 2 * t + 1) + lane * 16);
                ng_lds_read();
                if (!LAST) issue_w(i + CH + ch, ch, t);
                if (live) {                                // (a chunk's eight first, then its sum: shorter chains of roundings)
                    const int k = ACT ? 2 * (ch % 4) : 0;
                    acc[2 * t] += dot8(w0, a[k], a[k + 1], 0.f);
                    acc[2 * t + 1] += dot8(w1, a[k], a[k + 1], 0.f);
                }
            }
        }
    }
    __device__ __forceinline__ void run()
    {
        const int n = p0.n;
        if (n == 0) return;
        if (n <= CH) { stage<kOnly>(0); return; }
        int i = 0;
        for (; i + CH < n; i += CH) stage<kSteady>(i);
        stage<kLast>(i);
    }
    // the sums of the wavefront's columns, row by row
    __device__ __forceinline__ void leave(float *red, int wave) const
    {
#pragma unroll
        for (int o = 0; o < 2 * T; ++o) {
            float v = acc[o];
            v += dpp_mov<kDppXor1>(v);
            v += dpp_mov<kDppXor2>(v);
            v += dpp_mov<kDppHalfMirror>(v);
            if ((lane & 7) == 0) red[wave * 16 * T + 8 * o + (lane >> 3)] = v;
        }
    }
    // row `row` of W wavefronts' sums, in order
    template <int W>
    static __device__ __forceinline__ float total(const float *red, int row)
    {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) s += red[w * 16 * T + row];
        return s;
    }
};

// LayerNorm of one token, dealt like the stream: a wavefront has the x, gamma and beta of its own columns, at most 512; mean and
// squared deviations are joined over the W wavefronts in order, one behind the other (two passes over registers).
constexpr int kLoneX = 2048, kLoneVec = 1024;              // bytes of a wavefront's x (then its normalised columns), gamma, beta
constexpr int kLoneNorm = kLoneX + 2 * kLoneVec;
template <int W>
struct LoneNorm {
    char *vec, *mine;       // LDS: of all wavefronts, of this one
    int cn, lane, wave;
    bool half;              // x is fp16
    // four loads (where the wavefront has columns); columns: chunks [c0, c0 + cn) of 64
    __device__ __forceinline__ void request(char *lds, int c0, int cn_, const void *x, bool x_half, const __half *gamma, const __half *beta, int tid)
    {
        vec = lds; cn = cn_; half = x_half;
        lane = tid & 63; wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        mine = vec + wave * kLoneNorm;
        if (cn <= 0) return;
        const unsigned at = lds_address(mine), last = (unsigned)cn * 8u - 1u, p16 = min((unsigned)lane, last) * 16u;
        if (half) {                                        // (the second load has no purpose: the number of loads is fixed)
            const i32x4 rs = dma_rsrc(static_cast<const __half *>(x) + c0 * kNgChunk, (unsigned)cn * 128u);
            lds_dma16(rs, at, p16, 0u);
            lds_dma16(rs, at + 1024u, p16, 0u);
        } else {
            const i32x4 rs = dma_rsrc(static_cast<const float *>(x) + c0 * kNgChunk, (unsigned)cn * 256u);
            lds_dma16(rs, at, min((unsigned)lane, 2u * last + 1u) * 16u, 0u);
            lds_dma16(rs, at + 1024u, min((unsigned)lane + 64u, 2u * last + 1u) * 16u, 0u);
        }
        lds_dma16(dma_rsrc(gamma + c0 * kNgChunk, (unsigned)cn * 128u), at + kLoneX, p16, 0u);
        lds_dma16(dma_rsrc(beta + c0 * kNgChunk, (unsigned)cn * 128u), at + kLoneX + kLoneVec, p16, 0u);
    }
    // what request() asked for is there: the normalised columns in the place of x.  Two workgroup barriers.
    __device__ __forceinline__ void finish(int h, float eps)
    {
        float x[8];
        u32x4 g, b;
        {
            const bool real = lane < 8 * cn;               // this lane's 8 columns
            const char *at = mine + (half ? lane * 16 : lane * 32);
            const u32x4 xa = *reinterpret_cast<const u32x4 *>(at), xb = *reinterpret_cast<const u32x4 *>(half ? at : at + 16);
            g = *reinterpret_cast<const u32x4 *>(mine + kLoneX + lane * 16);
            b = *reinterpret_cast<const u32x4 *>(mine + kLoneX + kLoneVec + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 v = unpack_h2(xa[e]);
                const float lo = half ? v.x : __uint_as_float(e < 2 ? xa[2 * e] : xb[2 * e - 4]);
                const float hi = half ? v.y : __uint_as_float(e < 2 ? xa[2 * e + 1] : xb[2 * e - 3]);
                x[2 * e] = real ? lo : 0.f;
                x[2 * e + 1] = real ? hi : 0.f;
            }
        }
        auto stat = [&](int w) { return reinterpret_cast<float *>(vec + w * kLoneNorm + kLoneX); };
        auto joined = [&](float v, int slot) {             // sum over the workgroup, in order
            v = wave_sum(v);
            if (lane == 0) stat(wave)[slot] = v;
            __syncthreads();
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) t += stat(w)[slot];
            return t;
        };
        float s = 0.f, q = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += x[e];
        const float mean = joined(s, 0) / (float)h;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[e] -= mean;
            q += lane < 8 * cn ? x[e] * x[e] : 0.f;
        }
        const float inv = 1.0f / sqrtf(joined(q, 1) / (float)h + eps);
        float4 y[2];
        float *v = reinterpret_cast<float *>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 gg = unpack_h2(g[e]), bb = unpack_h2(b[e]);
            v[2 * e] = x[2 * e] * inv * gg.x + bb.x;
            v[2 * e + 1] = x[2 * e + 1] * inv * gg.y + bb.y;
        }
        float4 *to = reinterpret_cast<float4 *>(mine + lane * 32);
        to[0] = y[0]; to[1] = y[1];
        ng_lds_read();                                     // (only this wavefront reads them)
    }
};

}  // namespace cfpp
