// Projections of a layer for a single sequence (paper Sec. 2.2): the narrow products' arrangement (narrow_stream.h) with
// fp32 activations.
//
//   k_lone_in  : both LayerNorms, QKV rows + bias, rotary, K/V append, q; MLP-up rows + bias + GELU
//   k_lone_out : output projection and MLP-down as one product over the concatenated K, + biases + residual
//
// One token would fill two columns of a matrix instruction, and its heads and remainders in fp16 have fp16's range: a finite
// input whose gamma x or GELU(up) passes 65504 came out as NaN, and an element below 2^-3 lost bits.  A row of weights
// against fp32 values is eight fused multiply-adds a lane and KiB instead, a tenth of what the stream leaves time for, and the
// LayerNorm is applied ahead of the products: nothing is rounded to less than fp32 and nothing cancels behind them.
// A wavefront's part of x is 512 columns at most: its statistics take the time the first weights need to arrive.
// us a block of 1024 positions, heads and remainders through the matrix cores -> this: hidden 1280 24.2 -> 22.2, 2560 39.3 -> 37.5,
// 4096 74.6 -> 73.9; a layer of a stack: 512 16.4 -> 15.6, 1536 24.4 -> 22.7.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "narrow_stream.h"
#include "prefill_device.h"

namespace cfpp {

constexpr int kLoneWaves = 8, kLoneThreads = 64 * kLoneWaves;

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
    NgPiece p0, p1;
    const void *act;        // ACT: what the resource of the activations starts at
    unsigned act_bytes, act0, act1;        // its size; where the activations of each matrix's first column lie in it
    unsigned ring;          // LDS address of this wavefront's ring
    const char *mem;        // the same as a pointer
    const float *y;         // !ACT: this wavefront's activations
    int lane, octets, tail; // whole 8-row groups, rows beyond them
    float acc[2 * T];       // this lane's columns of row lane / 8 of each group

    static constexpr unsigned place_w(int ch, int o) { return (unsigned)((ACT ? ch / 4 + 1 : 0) + ch * PER + o) * 1024u; }
    static constexpr unsigned place_a(int quad) { return (unsigned)(quad * (1 + 4 * PER)) * 1024u; }

    __device__ __forceinline__ void issue_a(int i, int quad) const
    {
        const int k = i + (lane >> 4), c = k < p0.n ? p0.c0 + k : p1.c0 + k - p0.n;
        const unsigned v = (k < p0.n ? act0 : act1) + (unsigned)c * 256u + (unsigned)(lane & 15) * 16u;
        lds_dma16(dma_rsrc(act, act_bytes), ring + place_a(quad), k < p0.n + p1.n ? v : 0u, 0u);
    }
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
            if (ch >= p0.n + p1.n) break;                  // (uniform)
            if (ACT && ch % 4 == 0) issue_a(ch, ch / 4);
#pragma unroll
            for (int t = 0; t < T; ++t) issue_w(ch, ch, t);
        }
    }
    // what was requested ahead of begin() is there (!ACT: begin() requested whole chunks, CH or as many as there are)
    template <int N = CH>
    __device__ __forceinline__ void wait_ahead() const
    {
        if (p0.n + p1.n >= N) ng_wait<N * PER>();
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
            const bool live = CH == 1 || i + ch < p0.n + p1.n;             // (uniform)
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
        const int n = p0.n + p1.n;
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
    static __device__ __forceinline__ float total(const float *red, int row)
    {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kLoneWaves; ++w) s += red[w * 16 * T + row];
        return s;
    }
};

// the position, if it is inside the cache (uniform over the grid)
__device__ __forceinline__ bool lone_position_ok(const NarrowParams &P, int *pos)
{
    typedef const __attribute__((address_space(4))) int *Scalar;
    const int p = *(Scalar)reinterpret_cast<unsigned long long>(P.pos);
    const bool ok = p >= 0 && p < P.dm.max_seq;
    if (!ok && threadIdx.x == 0 && blockIdx.x == 0)
        __hip_atomic_store(&P.sync[kSyncErr], (unsigned)kErrBadPos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *pos = ok ? p : 0;
    return ok;
}

// A chunk to a stage, or as many as keep 8 KiB of a wavefront's weights in flight.
template <int T>
constexpr int lone_chunks() { return T == 1 ? 4 : T == 2 ? 2 : 1; }
constexpr int kLoneX = 2048, kLoneVec = 1024;              // bytes of a wavefront's x (then y), gamma, beta
template <int T>
constexpr int lone_in_lds() { return kLoneWaves * (LoneStream<T, lone_chunks<T>(), false>::kStage + kLoneX + 2 * kLoneVec); }

// LayerNorms, QKV rows and MLP-up rows.  Workgroups 0 .. wgs_q - 1 have P.rows rows each of the QKV matrix (even: a rotary
// pair stays in one), the others of the MLP-up matrix.  A wavefront has the x, gamma and beta of its own columns; mean and
// squared deviations are joined over the wavefronts in order, one behind the other (two passes over registers).
// LDS: rings (at the end: sums) | per wavefront x, gamma (then the statistics), beta.
template <int T>
__global__ void __launch_bounds__(kLoneThreads, 2) k_lone_in(NarrowParams P)
{
    using Stream = LoneStream<T, lone_chunks<T>(), false>;
    static_assert(lone_in_lds<T>() <= 160 * 1024, "");
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool up = (int)blockIdx.x >= P.wgs_q;
    const int r0 = ((int)blockIdx.x - (up ? P.wgs_q : 0)) * P.rows, rn = min(P.rows, (up ? f : 3 * h) - r0);
    // the epilogue's row (MLP-up) or row pair (QKV) of this thread, and its biases: requested ahead of the weights
    const int e0 = up ? min(tid, rn - 1) : min(2 * tid, rn - 2);
    const __half *bias = P.w + (up ? P.lay.b_up : P.lay.b_qkv) + r0;
    const __half k0 = bias[e0], k1 = bias[up ? e0 : e0 + 1];
    const int C = h / kNgChunk, c0 = C * wave / kLoneWaves, cn = C * (wave + 1) / kLoneWaves - c0;    // (hidden <= 4096: cn <= 8)
    char *vec = ng_lds + kLoneWaves * Stream::kStage, *mine = vec + wave * (kLoneX + 2 * kLoneVec);
    Stream st;
    st.p0.w = P.w + (up ? P.lay.w_up : P.lay.w_qkv) + (size_t)r0 * h;
    st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.c0 = c0; st.p0.n = cn;
    st.p1 = st.p0; st.p1.n = 0;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = ng_lds + wave * Stream::kStage;
    st.y = reinterpret_cast<const float *>(mine);
    if (cn > 0) {
        const unsigned at = lds_address(mine), last = (unsigned)cn * 8u - 1u, p16 = min((unsigned)lane, last) * 16u;
        if (P.layer == 0) {                                // (the second load has no purpose: the number of loads is fixed)
            const i32x4 rs = dma_rsrc(P.x_in + c0 * kNgChunk, (unsigned)cn * 128u);
            lds_dma16(rs, at, p16, 0u);
            lds_dma16(rs, at + 1024u, p16, 0u);
        } else {
            const i32x4 rs = dma_rsrc(P.xres + (size_t)((P.layer - 1) & 1) * h + c0 * kNgChunk, (unsigned)cn * 256u);
            lds_dma16(rs, at, min((unsigned)lane, 2u * last + 1u) * 16u, 0u);
            lds_dma16(rs, at + 1024u, min((unsigned)lane + 64u, 2u * last + 1u) * 16u, 0u);
        }
        lds_dma16(dma_rsrc(P.w + (up ? P.lay.ln2_g : P.lay.ln1_g) + c0 * kNgChunk, (unsigned)cn * 128u), at + kLoneX, p16, 0u);
        lds_dma16(dma_rsrc(P.w + (up ? P.lay.ln2_b : P.lay.ln1_b) + c0 * kNgChunk, (unsigned)cn * 128u), at + kLoneX + kLoneVec, p16, 0u);
    }
    st.begin(rn, tid);
    int pos;
    const bool ok = lone_position_ok(P, &pos);
    // rotary pair of this thread (QKV): head, part (q, k, v), dimension
    const int pk = r0 + e0, pd = pk / dm.d, i = pk - pd * dm.d, nh = pd / 3, c = pd - 3 * nh;
    const bool rot = !up && c < 2 && i < dm.r;
    st.wait_ahead();                                       // x, gamma and beta are there
    float x[8];
    u32x4 g, b;
    {
        const bool real = lane < 8 * cn;                   // this lane's 8 columns
        const char *at = mine + (P.layer == 0 ? lane * 16 : lane * 32);
        const u32x4 xa = *reinterpret_cast<const u32x4 *>(at), xb = *reinterpret_cast<const u32x4 *>(P.layer == 0 ? at : at + 16);
        g = *reinterpret_cast<const u32x4 *>(mine + kLoneX + lane * 16);
        b = *reinterpret_cast<const u32x4 *>(mine + kLoneX + kLoneVec + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 v = unpack_h2(xa[e]);
            const float lo = P.layer == 0 ? v.x : __uint_as_float(e < 2 ? xa[2 * e] : xb[2 * e - 4]);
            const float hi = P.layer == 0 ? v.y : __uint_as_float(e < 2 ? xa[2 * e + 1] : xb[2 * e - 3]);
            x[2 * e] = real ? lo : 0.f;
            x[2 * e + 1] = real ? hi : 0.f;
        }
    }
    auto stat = [&](int w) { return reinterpret_cast<float *>(vec + w * (kLoneX + 2 * kLoneVec) + kLoneX); };
    auto joined = [&](float v, int slot) {                 // sum over the workgroup, in order
        v = wave_sum(v);
        if (lane == 0) stat(wave)[slot] = v;
        __syncthreads();
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < kLoneWaves; ++w) t += stat(w)[slot];
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
    const float inv = 1.0f / sqrtf(joined(q, 1) / (float)h + dm.ln_eps);
    {
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
    const float2 cs = P.rope[rot ? (size_t)pos * (dm.r >> 1) + (i >> 1) : 0];
    st.run();
    __syncthreads();                                       // the rings have been read
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave(red, wave);
    __syncthreads();
    if (!ok) return;
    if (up) {
        if (tid < rn) P.m32[r0 + tid] = pf_gelu(Stream::total(red, tid) + __half2float(k0), dm.flags);
        return;
    }
    if (2 * tid >= rn) return;
    float v0 = Stream::total(red, 2 * tid) + __half2float(k0), v1 = Stream::total(red, 2 * tid + 1) + __half2float(k1);
    int d0 = i, d1 = i + 1;
    if (rot) {
        const float lo = v0 * cs.x - v1 * cs.y, hi = v1 * cs.x + v0 * cs.y;
        v0 = lo; v1 = hi;
        d0 = i >> 1; d1 = (i >> 1) + (dm.r >> 1);
    }
    if (c == 0) {
        P.q[nh * dm.d + d0] = v0;
        P.q[nh * dm.d + d1] = v1;
    } else {
        P.kv[kv_offset(dm, c - 1, P.kv_b0, nh, d0, pos)] = __float2half_rn(v0);
        P.kv[kv_offset(dm, c - 1, P.kv_b0, nh, d1, pos)] = __float2half_rn(v1);
    }
}

// Output projection and MLP-down as one product over the concatenated K ([attention | GELU(up)] . [W_dense | W_down]^T),
// + biases + residual.  A workgroup has at most 16 rows; a wavefront an eighth of the K values, with their activations.
// Four chunks to a stage, 8 KiB of weights a wavefront in flight: with eight a block takes 1.1 us more at hidden 2560, 0.9 at 4096.
using LoneOut = LoneStream<1, 4, true>;
constexpr int lone_out_lds() { return kLoneWaves * LoneOut::kStage; }
__global__ void __launch_bounds__(kLoneThreads, 2) k_lone_out(NarrowParams P)
{
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = (int)blockIdx.x * P.rows, rn = min(P.rows, h - r0), row = min(tid, rn - 1);
    const __half de = P.w[P.lay.b_dense + r0 + row], dn = P.w[P.lay.b_down + r0 + row];
    const float x = P.layer == 0 ? __half2float(P.x_in[r0 + row]) : P.xres[(size_t)((P.layer - 1) & 1) * h + r0 + row];
    const int C0 = h / kNgChunk, C = (h + f) / kNgChunk, c0 = C * wave / kLoneWaves, c1 = C * (wave + 1) / kLoneWaves;
    LoneOut st;
    st.p0.w = P.w + P.lay.w_dense + (size_t)r0 * h; st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.c0 = c0; st.p0.n = max(0, min(c1, C0) - c0);
    st.p1.w = P.w + P.lay.w_down + (size_t)r0 * f; st.p1.row_bytes = (unsigned)f * 2u;
    st.p1.c0 = max(0, c0 - C0); st.p1.n = max(0, c1 - max(c0, C0));
    st.act = P.m32;                                          // (the workspace, of at most 64 sequences, has the attention output behind GELU(up))
    st.act0 = (unsigned)((const char *)P.o32 - (const char *)P.m32); st.act1 = 0u;
    st.act_bytes = st.act0 + (unsigned)h * 4u;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * LoneOut::kStage);
    st.mem = ng_lds + wave * LoneOut::kStage;
    st.y = nullptr;
    st.begin(rn, tid);
    int pos;
    const bool ok = lone_position_ok(P, &pos);
    st.run();
    __syncthreads();
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave(red, wave);
    __syncthreads();
    if (!ok || tid >= rn) return;
    const float res = x + ((LoneOut::total(red, row) + __half2float(de)) + __half2float(dn));
    if (P.layer == P.n_layers - 1) P.out[r0 + row] = __float2half_rn(res);
    else P.xres[(size_t)(P.layer & 1) * h + r0 + row] = res;
}

// ---------------------------------------------------------------------------
template <int T>
static hipError_t lone_launch_in(const NarrowParams &P, int wgs, hipStream_t s)
{
    hipLaunchKernelGGL(k_lone_in<T>, dim3(wgs), dim3(kLoneThreads), lone_in_lds<T>(), s, P);
    return hipGetLastError();
}
hipError_t launch_lone_in(NarrowParams P, int grid, hipStream_t s)
{
    int wgs;
    P.rows = ng_in_rows(P.dm, grid, &P.wgs_q, &wgs);
    if (P.rows == 0) return hipErrorInvalidValue;
    switch ((P.rows + 15) / 16) {
    case 1: return lone_launch_in<1>(P, wgs, s);
    case 2: return lone_launch_in<2>(P, wgs, s);
    case 3: return lone_launch_in<3>(P, wgs, s);
    case 4: case 5: return lone_launch_in<5>(P, wgs, s);
    case 6: case 7: return lone_launch_in<7>(P, wgs, s);
    }
    return lone_launch_in<8>(P, wgs, s);
}

hipError_t launch_lone_out(NarrowParams P, int grid, hipStream_t s)
{
    P.rows = min(16, (P.dm.h + grid - 1) / grid);
    hipLaunchKernelGGL(k_lone_out, dim3((P.dm.h + P.rows - 1) / P.rows), dim3(kLoneThreads), lone_out_lds(), s, P);
    return hipGetLastError();
}

// allow more than the default 64 KiB of dynamic LDS
template <int T>
static hipError_t lone_prepare()
{
    return hipFuncSetAttribute((const void *)k_lone_in<T>, hipFuncAttributeMaxDynamicSharedMemorySize, lone_in_lds<T>());
}
hipError_t prepare_lone_kernels()
{
    hipError_t e;
    if ((e = lone_prepare<1>()) != hipSuccess || (e = lone_prepare<2>()) != hipSuccess || (e = lone_prepare<3>()) != hipSuccess ||
        (e = lone_prepare<5>()) != hipSuccess || (e = lone_prepare<7>()) != hipSuccess || (e = lone_prepare<8>()) != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_lone_out, hipFuncAttributeMaxDynamicSharedMemorySize, lone_out_lds());
}

}  // namespace cfpp
