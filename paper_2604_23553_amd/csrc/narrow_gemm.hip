// Projections of a layer for few tokens (paper Sec. 2.2): the sequences of a decode step, a group of prompt tokens; two to
// eight of them (one: lone_gemm.hip).  The weights are read once and their way from memory is what takes time, so everything here is arranged around that stream.
//
//   k_ng_in  : both LayerNorms, QKV rows + bias, rotary, K/V append, q; MLP-up rows + bias + GELU
//   k_ng_dense : output projection, + MLP-down's parts, which the attention launch leaves (narrow_attention.hip), + biases + residual
//
// How the weights are streamed: narrow_stream.h.
// Kernel times, 8 sequences, the kernels before (weights through registers, four rows to a load, activations of a
// workgroup in LDS) -> these: hidden 2560: k_ng_in 28.7 -> 17.5 us; output projection and MLP-down in one
// kernel 23.5 -> 15.2 (5 sequences) and 24.7 -> 17.3 (8), without MLP-down, which the attention launch has now, k_ng_dense is 6.3 and 6.8;
// hidden 4096: 49.1 -> 37.5, 43.6 -> 31.3 and 8.8.  k_ng_dense is a launch, a trip for the weights and one for the sums: 13 MB at hidden 2560.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "narrow_stream.h"
#include "prefill_device.h"

namespace cfpp {

constexpr int kNgWaves = 8, kNgThreads = 64 * kNgWaves;

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
constexpr int ng_in_lds() { return kNgWaves * (NgStream<T, 1, SRC, 1>::kStage + 1024 + kNgSet * 8); }

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
    using Stream = NgStream<T, 1, SRC, 1>;
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
    st.template leave<1>(red, wave, 0);
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
                split_half(pf_gelu((ng_total<kNgWaves>(red, Stream::kSetFloats, rr, b) - mean * k.x) * inv + k.y, dm.flags), hi, lo);
                const size_t at = ng_at(b, r0 + rr, f, P.nt);
                P.m[at] = hi; P.m[at + 8 * P.nt] = lo;
            }
        }
        return;
    }
    if (2 * row >= rn) return;
    const float2 s = ng_total2<kNgWaves>(red, Stream::kSetFloats, 2 * row, b);
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

// Output projection, + MLP-down's parts (narrow_attention.hip) + biases + residual.  A workgroup has at most 16 rows; a
// wavefront an eighth of the K values.
constexpr int kNgDenseChunks = 3;
constexpr int ng_dense_lds() { return kNgWaves * NgStream<1, 1, kNgPlanes, kNgDenseChunks>::kStage; }
__global__ void __launch_bounds__(kNgThreads, 2) k_ng_dense(NarrowParams P)
{
    using Stream = NgStream<1, 1, kNgPlanes, kNgDenseChunks>;
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = (int)blockIdx.x * P.rows, rn = min(P.rows, h - r0);
    const int b = tid & (kNgSet - 1), row = min(tid >> 3, rn - 1);
    const __half de = P.w[P.lay.b_dense + r0 + row], dn = P.w[P.lay.b_down + r0 + row];
    const int xb = min(b, P.n - 1);                        // the layer input, fp16 or fp32 (converted when the weights are through)
    const __half x16 = P.x_in[(size_t)xb * h + r0 + row];
    const float x32 = P.xres[((size_t)xb * 2 + ((P.layer - 1) & 1)) * h + r0 + row];
    float down[kDownParts];
    down_parts(P, xb, r0 + row, down);
    const int C = h / kNgChunk, c0 = C * wave / kNgWaves;
    Stream st;
    st.p0.w = P.w + P.lay.w_dense + (size_t)r0 * h; st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.b = P.o; st.p0.b_bytes = (unsigned)P.nt * (unsigned)h * 4u;
    st.p0.c0 = c0; st.p0.n = C * (wave + 1) / kNgWaves - c0;
    st.p1 = st.p0; st.p1.n = 0;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = ng_lds + wave * Stream::kStage;
    st.gamma = nullptr;
    st.begin(rn, P.n, P.nt, 0u, tid);
    int pos;
    const bool ok = ng_positions_ok(P, b, &pos);
    st.run();
    __syncthreads();
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave<1>(red, wave, 0);
    __syncthreads();
    if (!ok || b >= P.n || (tid >> 3) >= rn) return;
    const float x = P.layer == 0 ? __half2float(x16) : x32;
    const float res = x + (((ng_total<kNgWaves>(red, Stream::kSetFloats, row, b) + down_sum(P, down)) + __half2float(de)) + __half2float(dn));
    if (P.layer == P.n_layers - 1) P.out[(size_t)b * h + r0 + row] = __float2half_rn(res);
    else P.xres[((size_t)b * 2 + (P.layer & 1)) * h + r0 + row] = res;
}

// ---------------------------------------------------------------------------
// Shapes and launch options that run the batched path: a wavefront's part of gamma (x) is 512 columns at most, a workgroup of the
// first product has up to kNgTileMax tiles of rows.  (An MLP that is no multiple of hidden keeps to the phase kernels.)
bool bat_supported(const Dims &dm, int grid, int threads)
{
    int wgs_q, wgs;
    return threads == kNgThreads && grid >= 1 && dm.h % 128 == 0 && dm.f % dm.h == 0 && dm.h <= 4096 &&
           ng_in_rows(dm, grid, &wgs_q, &wgs) > 0;
}

template <int T>
static hipError_t ng_launch_in(const NarrowParams &P, int wgs, hipStream_t s)
{
    if (P.layer == 0) hipLaunchKernelGGL((k_ng_in<T, kNgRaw16>), dim3(wgs), dim3(kNgThreads), (ng_in_lds<T, kNgRaw16>()), s, P);
    else hipLaunchKernelGGL((k_ng_in<T, kNgRaw32>), dim3(wgs), dim3(kNgThreads), (ng_in_lds<T, kNgRaw32>()), s, P);
    return hipGetLastError();
}

hipError_t launch_bat_in(NarrowParams P, int grid, hipStream_t s)
{
    int wgs;
    P.rows = ng_in_rows(P.dm, grid, &P.wgs_q, &wgs);
    if (P.rows == 0) return hipErrorInvalidValue;
    const int t = (P.rows + 15) / 16;
    if (t <= 1) return ng_launch_in<1>(P, wgs, s);
    if (t <= 2) return ng_launch_in<2>(P, wgs, s);
    if (t <= 3) return ng_launch_in<3>(P, wgs, s);
    if (t <= 5) return ng_launch_in<5>(P, wgs, s);
    return ng_launch_in<8>(P, wgs, s);
}

hipError_t launch_bat_dense(NarrowParams P, int grid, hipStream_t s)
{
    P.rows = min(16, (P.dm.h + grid - 1) / grid);
    hipLaunchKernelGGL(k_ng_dense, dim3((P.dm.h + P.rows - 1) / P.rows), dim3(kNgThreads), ng_dense_lds(), s, P);
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
    return hipFuncSetAttribute((const void *)k_ng_dense, hipFuncAttributeMaxDynamicSharedMemorySize, ng_dense_lds());
}

}  // namespace cfpp
