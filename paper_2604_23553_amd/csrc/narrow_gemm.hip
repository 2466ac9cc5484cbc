// Projections of a layer for few tokens (paper Sec. 2.2): the sequences of a decode step, a group of prompt tokens.  The
// weights are read once and their way from memory is what takes time, so everything here is arranged around that stream.
//
//   k_ng_in  : both LayerNorms, QKV rows + bias, rotary, K/V append, q; MLP-up rows + bias + GELU
//   k_ng_out : output projection and MLP-down as one product over the concatenated K, + biases + residual
//
// A workgroup (8 wavefronts, one to a CU) owns a contiguous range of rows of one matrix and its wavefronts split K: a
// wavefront streams its columns of all rows, 64 columns (a chunk: whole 128-byte lines) at a time, through an LDS ring of its
// own that is filled by memory-to-LDS loads.  No wavefront waits for another before the sums are added, no register
// holds what is in flight, and a row counts for nothing but its own bytes, whatever their number.  Measured with loads alone
// (one launch, launch included): 92 MB of 17920 x 2560: 15.7 us, 235 MB of 28672 x 4096: 36 us = 6.5 TB/s.
// Kernel times, 8 sequences, the kernels before (weights through registers, four rows to a load, activations of a
// workgroup in LDS) -> these: hidden 2560: k_ng_in 28.7 -> 17.5 us, k_ng_out 23.5 -> 15.2 (5 sequences) and 24.7 -> 17.8 (8);
// hidden 4096: 49.0 -> 39.6, 42.8 -> 32.8.  What is left of k_ng_out beyond its weights (13 us at 2560) is the activations:
// every workgroup reads all of them from the L2, 8 tokens 410 KB beside 256 KB of weights.
//
// v_mfma_f32_16x16x32_f16: A = 16 rows x 32 columns of weights, from the ring; B = the same 32 columns of 8 tokens, the
// fp16 heads of their fp32 activations in columns 0..7 and the remainders in 8..15 (y = hi + lo to ~2^-22): one
// instruction per KiB of weights.  The two columns of a token and the 8 wavefronts' parts of K are added in a fixed
// order at the end: one bit pattern per build.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "device_utils.h"
#include "half_split.h"
#include "lds_dma.h"
#include "narrow_params.h"
#include "prefill_device.h"

namespace cfpp {

typedef _Float16 ng_f16x8 __attribute__((ext_vector_type(8)));

constexpr int kNgWaves = 8, kNgThreads = 64 * kNgWaves, kNgChunk = 64, kNgTileMax = 8;
// what the activations are in memory: planes (ng_at), or the layer input itself (fp32 or fp16), which the
// wavefronts multiply by gamma and split on the way
enum { kNgPlanes, kNgRaw32, kNgRaw16 };

// chunks [c0, c0 + n) of a workgroup's rows of one matrix, and where their activations are
struct NgPiece {
    const void *w, *b;      // first row; activations
    unsigned row_bytes, b_bytes;
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

// The stream of one wavefront.  A stage is CH chunks; of each, NB loads bring the activations and 2 T the weights of
// T tiles of 16 rows (a load: 8 rows x 128 bytes).  Every load of a stage has its place in the ring, and is requested
// again - for the next stage - as soon as what it brought has been read: NI - 2 or NI - NB loads are always in
// flight behind the one that is waited for, by count.  Loads without a purpose (rows past the last, chunks past
// the end) read one line over and over.
template <int T, int SRC, int CH>
struct NgStream {
    static constexpr int NB = SRC == kNgRaw16 ? 1 : 2, PER = NB + 2 * T, NI = CH * PER, kStage = NI * 1024;
    static_assert(NI <= 62, "the memory counter's range");
    NgPiece p0, p1;
    unsigned ring;          // LDS address of this wavefront's ring
    const char *mem;        // the same as a pointer
    const char *gamma;      // this wavefront's columns of gamma in LDS (layer input only)
    int lane, octets, tail; // whole 8-row groups, rows beyond them
    unsigned v_b, place, a_at;
    f32x4 acc[T];
    float mean, m2;         // of the layer input's columns this lane has seen

    __device__ __forceinline__ void issue_b(int i, int ch) const
    {
        const bool second = i >= p0.n, live = i < p0.n + p1.n;
        const int c = second ? p1.c0 + i - p0.n : p0.c0 + i;
        const i32x4 rs = dma_rsrc(second ? p1.b : p0.b, second ? p1.b_bytes : p0.b_bytes);
#pragma unroll
        for (int k = 0; k < NB; ++k)
            lds_dma16(rs, ring + (unsigned)(ch * PER + k) * 1024u, live ? v_b : 0u, live ? (unsigned)(NB * c + k) * b_step() : 0u);
    }
    unsigned b_block;       // planes: bytes of a block of 32 columns
    __device__ __forceinline__ unsigned b_step() const { return SRC == kNgPlanes ? b_block : 128u; }

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
        for (int t = 0; t < T; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
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
    __device__ __forceinline__ void activations(int i, int ch, ng_f16x8 (&b)[2])
    {
        const char *at = mem + ch * PER * 1024;
        if (SRC == kNgPlanes) {
#pragma unroll
            for (int k = 0; k < 2; ++k) b[k] = *reinterpret_cast<const ng_f16x8 *>(at + k * 1024 + lane * 16);
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
            ng_f16x8 b[2];
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
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w0, b[0], acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1, b[1], acc[t], 0, 0, 0);
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

    // the sums of the wavefront's tiles, rows side by side: kNgRedCol floats per column
    __device__ __forceinline__ void leave(float *red, int wave) const
    {
        const int col = lane & 15, r4 = 4 * (lane >> 4);
#pragma unroll
        for (int t = 0; t < T; ++t) *reinterpret_cast<f32x4 *>(red + ((wave * T + t) * 16 + col) * 20 + r4) = acc[t];
    }
};

// row `row` of the workgroup for token b (of a set): heads' and remainders' columns of the 8 wavefronts, in order
template <int T>
__device__ __forceinline__ float ng_total(const float *red, int row, int b)
{
    const float *p = red + ((row >> 4) * 16 + b) * 20 + (row & 15);
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kNgWaves; ++w) s += p[w * T * 320] + p[w * T * 320 + 160];
    return s;
}
template <int T>
__device__ __forceinline__ float2 ng_total2(const float *red, int row, int b)         // rows row, row + 1 (row even)
{
    const float *p = red + ((row >> 4) * 16 + b) * 20 + (row & 15);
    float2 s{0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kNgWaves; ++w) {
        const float2 h = *reinterpret_cast<const float2 *>(p + w * T * 320), l = *reinterpret_cast<const float2 *>(p + w * T * 320 + 160);
        s.x += h.x + l.x; s.y += h.y + l.y;
    }
    return s;
}

// All positions inside the cache?  (uniform over the grid.)  pos: that of token b.  Scalar loads: a vector load behind the
// stream's first requests would have to wait for them.
__device__ __forceinline__ bool ng_positions_ok(const NarrowParams &P, int b, int *pos)
{
    typedef const __attribute__((address_space(4))) int *Scalar;
    const Scalar at = (Scalar)reinterpret_cast<unsigned long long>(P.pos);
    bool ok = true;
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kNgSet; ++i) {
        const int p = at[min(i, P.n - 1)];
        ok = ok && p >= 0 && p < P.dm.max_seq;
        mine = i == b ? p : mine;
    }
    if (!ok && threadIdx.x == 0 && blockIdx.x == 0)
        __hip_atomic_store(&P.sync[kSyncErr], (unsigned)kErrBadPos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *pos = ok ? mine : 0;
    return ok;
}

template <int T, int SRC>
constexpr int ng_in_lds() { return kNgWaves * (NgStream<T, SRC, 1>::kStage + 1024 + kNgSet * 8); }

// LayerNorms, QKV rows and MLP-up rows.  Workgroups 0 .. wgs_q - 1 have P.rows rows each of the QKV matrix (even: a rotary
// pair stays in one), the others of the MLP-up matrix: a workgroup needs one LayerNorm's input.  The statistics are not waited
// for: the matrices run on gamma * x and the epilogue completes
//   W (gamma (x - mu) inv + beta) + b = inv (W (gamma x) - mu s) + c
// with s = W gamma and c = W beta + b from the packing (PackedLayout::rc_qkv, rc_up).  Mean and variance come from the
// columns that pass by: 16 of a token at a time, their mean and squared deviations joined pairwise.
// LDS: rings (at the end: sums) | gamma | statistics.
template <int T, int SRC>
__global__ void __launch_bounds__(kNgThreads, 2) k_ng_in(NarrowParams P)
{
    using Stream = NgStream<T, SRC, 1>;
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool up = (int)blockIdx.x >= P.wgs_q;
    const int r0 = ((int)blockIdx.x - (up ? P.wgs_q : 0)) * P.rows, rn = min(P.rows, (up ? f : 3 * h) - r0);
    const int b = tid & (kNgSet - 1), row = tid >> 3;      // the epilogue's token; its row (MLP-up: and row + 64) or row pair
    // what the epilogue needs of memory: requested ahead of the weights
    const float2 *rc = reinterpret_cast<const float2 *>(P.w + (up ? P.lay.rc_up : P.lay.rc_qkv)) + r0;
    const int e0 = up ? min(row, rn - 1) : min(2 * row, rn - 2), e1 = up ? min(row + 64, rn - 1) : e0 + 1;
    const float2 k0 = rc[e0], k1 = rc[e1];
    char *gam = ng_lds + kNgWaves * Stream::kStage + wave * 1024;
    float2 *stat = reinterpret_cast<float2 *>(ng_lds + kNgWaves * (Stream::kStage + 1024));
    Stream st;
    const int C = h / kNgChunk, c0 = C * wave / kNgWaves, cn = C * (wave + 1) / kNgWaves - c0;
    st.p0.w = P.w + (up ? P.lay.w_up : P.lay.w_qkv) + (size_t)r0 * h;
    st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.b = SRC == kNgRaw16 ? (const void *)P.x_in : (const void *)(P.xres + (size_t)((P.layer - 1) & 1) * h);
    const unsigned x_stride = SRC == kNgRaw16 ? (unsigned)h * 2u : (unsigned)h * 8u;
    st.p0.b_bytes = (unsigned)(P.n - 1) * x_stride + (unsigned)h * (SRC == kNgRaw16 ? 2u : 4u);
    st.p0.c0 = c0; st.p0.n = cn;
    st.p1 = st.p0; st.p1.n = 0;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = ng_lds + wave * Stream::kStage;
    st.gamma = gam;
    // gamma of this wavefront's columns (at most 512): one load
    if (cn > 0)
        lds_dma16(dma_rsrc(P.w + (up ? P.lay.ln2_g : P.lay.ln1_g) + c0 * kNgChunk, (unsigned)cn * 128u), lds_address(gam), (unsigned)min(lane, cn * 8 - 1) * 16u, 0u);
    st.begin(rn, P.n, P.nt, x_stride, tid);
    int pos;
    const bool ok = ng_positions_ok(P, b, &pos);
    // rotary pair of this thread (QKV): head, part (q, k, v), dimension
    const int pk = r0 + e0, pd = pk / dm.d, i = pk - pd * dm.d, nh = pd / 3, c = pd - 3 * nh;
    const bool rot = !up && c < 2 && i < dm.r;
    const float2 cs = P.rope[rot ? (size_t)pos * (dm.r >> 1) + (i >> 1) : 0];
    st.run();
    // statistics of the wavefront's columns: the four lane groups' joined (equal counts), one value a token
    {
        float mean = st.mean, m2 = st.m2, n = 16.f * (float)cn;
#pragma unroll
        for (int x = 16; x <= 32; x *= 2) {
            const float om = __shfl_xor(mean, x, 64), oq = __shfl_xor(m2, x, 64), dl = om - mean;
            mean = 0.5f * (mean + om);
            m2 = (m2 + oq) + dl * dl * (0.5f * n);
            n *= 2.f;
        }
        if (lane < kNgSet) stat[wave * kNgSet + lane] = float2{mean, m2};
    }
    __syncthreads();                                       // the rings have been read
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave(red, wave);
    __syncthreads();
    if (!ok || b >= P.n) return;
    float mean = 0.f, m2 = 0.f;
#pragma unroll
    for (int w = 0; w < kNgWaves; ++w) mean = fmaf((float)(C * (w + 1) / kNgWaves - C * w / kNgWaves), stat[w * kNgSet + b].x, mean);
    mean /= (float)C;
#pragma unroll
    for (int w = 0; w < kNgWaves; ++w) {
        const float2 s = stat[w * kNgSet + b];
        const float dl = s.x - mean;
        m2 += fmaf(dl * dl, (float)((C * (w + 1) / kNgWaves - C * w / kNgWaves) * kNgChunk), s.y);
    }
    const float inv = 1.0f / sqrtf(m2 / (float)h + dm.ln_eps);
    if (up) {
#pragma unroll
        for (int j = 0; j < (T > 4 ? 2 : 1); ++j) {
            const int rr = row + 64 * j;
            if (rr < rn) {
                const float2 k = j ? k1 : k0;
                __half hi, lo;
                split_half(pf_gelu((ng_total<T>(red, rr, b) - mean * k.x) * inv + k.y, dm.flags), hi, lo);
                const size_t at = ng_at(b, r0 + rr, f, P.nt);
                P.m[at] = hi; P.m[at + 8 * P.nt] = lo;
            }
        }
        return;
    }
    if (2 * row >= rn) return;
    const float2 s = ng_total2<T>(red, 2 * row, b);
    float v0 = (s.x - mean * k0.x) * inv + k0.y, v1 = (s.y - mean * k1.x) * inv + k1.y;
    int d0 = i, d1 = i + 1;
    if (rot) {
        const float lo = v0 * cs.x - v1 * cs.y, hi = v1 * cs.x + v0 * cs.y;
        v0 = lo; v1 = hi;
        d0 = i >> 1; d1 = (i >> 1) + (dm.r >> 1);
    }
    if (c == 0) {
        P.q[(size_t)b * h + nh * dm.d + d0] = v0;
        P.q[(size_t)b * h + nh * dm.d + d1] = v1;
    } else {
        P.kv[kv_offset(dm, c - 1, P.kv_b0 + b * P.kv_bstep, nh, d0, pos)] = __float2half_rn(v0);
        P.kv[kv_offset(dm, c - 1, P.kv_b0 + b * P.kv_bstep, nh, d1, pos)] = __float2half_rn(v1);
    }
}

// Output projection and MLP-down as one product over the concatenated K ([attention | GELU(up)] . [W_dense | W_down]^T),
// + biases + residual.  A workgroup has at most 16 rows; a wavefront an eighth of the K values.
constexpr int kNgOutChunks = 3;
constexpr int ng_out_lds() { return kNgWaves * NgStream<1, kNgPlanes, kNgOutChunks>::kStage; }
__global__ void __launch_bounds__(kNgThreads, 2) k_ng_out(NarrowParams P)
{
    using Stream = NgStream<1, kNgPlanes, kNgOutChunks>;
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = (int)blockIdx.x * P.rows, rn = min(P.rows, h - r0);
    const int b = tid & (kNgSet - 1), row = min(tid >> 3, rn - 1);
    const __half de = P.w[P.lay.b_dense + r0 + row], dn = P.w[P.lay.b_down + r0 + row];
    const int xb = min(b, P.n - 1);                        // the layer input, fp16 or fp32 (converted when the weights are through)
    const __half x16 = P.x_in[(size_t)xb * h + r0 + row];
    const float x32 = P.xres[((size_t)xb * 2 + ((P.layer - 1) & 1)) * h + r0 + row];
    const int C0 = h / kNgChunk, C = (h + f) / kNgChunk, c0 = C * wave / kNgWaves, c1 = C * (wave + 1) / kNgWaves;
    Stream st;
    st.p0.w = P.w + P.lay.w_dense + (size_t)r0 * h; st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.b = P.o; st.p0.b_bytes = (unsigned)P.nt * (unsigned)h * 4u;
    st.p0.c0 = c0; st.p0.n = max(0, min(c1, C0) - c0);
    st.p1.w = P.w + P.lay.w_down + (size_t)r0 * f; st.p1.row_bytes = (unsigned)f * 2u;
    st.p1.b = P.m; st.p1.b_bytes = (unsigned)P.nt * (unsigned)f * 4u;
    st.p1.c0 = max(0, c0 - C0); st.p1.n = max(0, c1 - max(c0, C0));
    st.ring = lds_address(ng_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = ng_lds + wave * Stream::kStage;
    st.gamma = nullptr;
    st.begin(rn, P.n, P.nt, 0u, tid);
    int pos;
    const bool ok = ng_positions_ok(P, b, &pos);
    st.run();
    __syncthreads();
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave(red, wave);
    __syncthreads();
    if (!ok || b >= P.n || (tid >> 3) >= rn) return;
    const float x = P.layer == 0 ? __half2float(x16) : x32;
    const float res = x + ((ng_total<1>(red, row, b) + __half2float(de)) + __half2float(dn));
    if (P.layer == P.n_layers - 1) P.out[(size_t)b * h + r0 + row] = __float2half_rn(res);
    else P.xres[((size_t)b * 2 + (P.layer & 1)) * h + r0 + row] = res;
}

// ---------------------------------------------------------------------------
// Rows of a workgroup such that the workgroups of both matrices come to at most one (or, where that would be more
// than kNgTileMax tiles of 16, a few) per CU; even.
static int ng_in_rows(const Dims &dm, int n_cu, int *wgs_q, int *wgs)
{
    for (int per = 1;; ++per) {
        for (int rows = 2; rows <= 16 * kNgTileMax; rows += 2) {
            const int q = (3 * dm.h + rows - 1) / rows, u = (dm.f + rows - 1) / rows;
            if (q + u <= per * n_cu) { *wgs_q = q; *wgs = q + u; return rows; }
        }
    }
}

// Shapes and launch options that run the batched path.  (The bounds on rows per workgroup and on LDS are those of the
// grid that the option names; the kernels here choose their own.)
bool bat_supported(const Dims &dm, int grid, int threads)
{
    if (threads != 512 || grid < 1 || dm.h % 128 != 0 || dm.f % dm.h != 0 || dm.h > 4096) return false;
    auto rows = [&](int n) { return (n + grid - 1) / grid; };
    auto rc = [](int n) { return (n + 3) & ~3; };
    const int rq = (rows(3 * dm.h) + 1) & ~1, ru = rows(dm.f), rh = rows(dm.h);
    const size_t act = (size_t)32 * (dm.h + 32), in = act + (132 + (size_t)64 * (rc(rq) + rc(ru))) * 4, out = act + (size_t)256 * rc(rh);
    return (ru > rq ? ru : rq) <= 64 && (in > out ? in : out) <= 160 * 1024 && (unsigned long long)packed_layout(dm.h, dm.f).total * 2 < (1ull << 32);
}

template <int T>
static hipError_t ng_launch_in(const NarrowParams &P, int wgs, hipStream_t s)
{
    if (P.layer == 0) hipLaunchKernelGGL((k_ng_in<T, kNgRaw16>), dim3(wgs), dim3(kNgThreads), (ng_in_lds<T, kNgRaw16>()), s, P);
    else hipLaunchKernelGGL((k_ng_in<T, kNgRaw32>), dim3(wgs), dim3(kNgThreads), (ng_in_lds<T, kNgRaw32>()), s, P);
    return hipGetLastError();
}

hipError_t launch_bat_in(NarrowParams P, int n_cu, hipStream_t s)
{
    int wgs;
    P.rows = ng_in_rows(P.dm, n_cu, &P.wgs_q, &wgs);
    const int t = (P.rows + 15) / 16;
    if (t <= 1) return ng_launch_in<1>(P, wgs, s);
    if (t <= 2) return ng_launch_in<2>(P, wgs, s);
    if (t <= 3) return ng_launch_in<3>(P, wgs, s);
    if (t <= 5) return ng_launch_in<5>(P, wgs, s);
    return ng_launch_in<8>(P, wgs, s);
}

hipError_t launch_bat_out(NarrowParams P, int n_cu, hipStream_t s)
{
    P.rows = min(16, (P.dm.h + n_cu - 1) / n_cu);
    hipLaunchKernelGGL(k_ng_out, dim3((P.dm.h + P.rows - 1) / P.rows), dim3(kNgThreads), ng_out_lds(), s, P);
    return hipGetLastError();
}

// allow more than the default 64 KiB of dynamic LDS
template <int T>
static hipError_t ng_prepare()
{
    const hipError_t e = hipFuncSetAttribute((const void *)k_ng_in<T, kNgRaw16>, hipFuncAttributeMaxDynamicSharedMemorySize, ng_in_lds<T, kNgRaw16>());
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_ng_in<T, kNgRaw32>, hipFuncAttributeMaxDynamicSharedMemorySize, ng_in_lds<T, kNgRaw32>());
}
hipError_t prepare_narrow_kernels()
{
    hipError_t e;
    if ((e = ng_prepare<1>()) != hipSuccess || (e = ng_prepare<2>()) != hipSuccess || (e = ng_prepare<3>()) != hipSuccess ||
        (e = ng_prepare<5>()) != hipSuccess || (e = ng_prepare<8>()) != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_ng_out, hipFuncAttributeMaxDynamicSharedMemorySize, ng_out_lds());
}

}  // namespace cfpp
