// Projections of a layer for a single sequence (paper Sec. 2.2): the narrow products' arrangement (narrow_stream.h) with
// fp32 activations.
//
//   k_lone_in  : both LayerNorms, QKV rows + bias, rotary, K/V append, q; MLP-up rows + bias + GELU
//   k_lone_dense : output projection, + MLP-down's parts, which the attention launch leaves (narrow_attention.hip), + biases + residual
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
#include "lone_stream.h"
#include "prefill_device.h"

namespace cfpp {

constexpr int kLoneWaves = 8, kLoneThreads = 64 * kLoneWaves;

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
template <int T>
constexpr int lone_in_lds() { return kLoneWaves * (LoneStream<T, lone_chunks<T>(), false>::kStage + kLoneNorm); }

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
    const int h = dm.h, f = dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool up = (int)blockIdx.x >= P.wgs_q;
    const int r0 = ((int)blockIdx.x - (up ? P.wgs_q : 0)) * P.rows, rn = min(P.rows, (up ? f : 3 * h) - r0);
    // the epilogue's row (MLP-up) or row pair (QKV) of this thread, and its biases: requested ahead of the weights
    const int e0 = up ? min(tid, rn - 1) : min(2 * tid, rn - 2);
    const __half *bias = P.w + (up ? P.lay.b_up : P.lay.b_qkv) + r0;
    const __half k0 = bias[e0], k1 = bias[up ? e0 : e0 + 1];
    const int C = h / kNgChunk, c0 = C * wave / kLoneWaves, cn = C * (wave + 1) / kLoneWaves - c0;    // (hidden <= 4096: cn <= 8)
    char *vec = ng_lds + kLoneWaves * Stream::kStage;
    Stream st;
    st.p0.w = P.w + (up ? P.lay.w_up : P.lay.w_qkv) + (size_t)r0 * h;
    st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.c0 = c0; st.p0.n = cn;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = ng_lds + wave * Stream::kStage;
    st.y = reinterpret_cast<const float *>(vec + wave * kLoneNorm);
    LoneNorm<kLoneWaves> norm;
    norm.request(vec, c0, cn, P.layer == 0 ? (const void *)P.x_in : (const void *)(P.xres + (size_t)((P.layer - 1) & 1) * h), P.layer == 0,
                 P.w + (up ? P.lay.ln2_g : P.lay.ln1_g), P.w + (up ? P.lay.ln2_b : P.lay.ln1_b), tid);
    st.begin(rn, tid);
    int pos;
    const bool ok = lone_position_ok(P, &pos);
    // rotary pair of this thread (QKV): head, part (q, k, v), dimension
    const int pk = r0 + e0, pd = pk / dm.d, i = pk - pd * dm.d, nh = pd / 3, c = pd - 3 * nh;
    const bool rot = !up && c < 2 && i < dm.r;
    st.wait_ahead();                                       // x, gamma and beta are there
    norm.finish(h, dm.ln_eps);
    const float2 cs = P.rope[rot ? (size_t)pos * (dm.r >> 1) + (i >> 1) : 0];
    st.run();
    __syncthreads();                                       // the rings have been read
    float *red = reinterpret_cast<float *>(ng_lds);
    st.leave(red, wave);
    __syncthreads();
    if (!ok) return;
    if (up) {
        if (tid < rn) P.m32[r0 + tid] = pf_gelu(Stream::template total<kLoneWaves>(red, tid) + __half2float(k0), dm.flags);
        return;
    }
    if (2 * tid >= rn) return;
    float v0 = Stream::template total<kLoneWaves>(red, 2 * tid) + __half2float(k0), v1 = Stream::template total<kLoneWaves>(red, 2 * tid + 1) + __half2float(k1);
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

// Output projection, + MLP-down's parts (narrow_attention.hip) + biases + residual.  A workgroup has at most 16 rows; a wavefront
// an eighth of the K values, with their activations.
using LoneDense = LoneStream<1, 4, true>;
constexpr int lone_dense_lds() { return kLoneWaves * LoneDense::kStage; }
__global__ void __launch_bounds__(kLoneThreads, 2) k_lone_dense(NarrowParams P)
{
    extern __shared__ __align__(16) char ng_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = (int)blockIdx.x * P.rows, rn = min(P.rows, h - r0), row = min(tid, rn - 1);
    const __half de = P.w[P.lay.b_dense + r0 + row], dn = P.w[P.lay.b_down + r0 + row];
    const float x = P.layer == 0 ? __half2float(P.x_in[r0 + row]) : P.xres[(size_t)((P.layer - 1) & 1) * h + r0 + row];
    float down[kDownParts];
    down_parts(P, 0, r0 + row, down);
    const int C = h / kNgChunk, c0 = C * wave / kLoneWaves;
    LoneDense st;
    st.p0.w = P.w + P.lay.w_dense + (size_t)r0 * h; st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.c0 = c0; st.p0.n = C * (wave + 1) / kLoneWaves - c0;
    st.act = P.o32;
    st.act_bytes = (unsigned)h * 4u;
    st.ring = lds_address(ng_lds) + (unsigned)(wave * LoneDense::kStage);
    st.mem = ng_lds + wave * LoneDense::kStage;
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
    const float res = x + (((LoneDense::total<kLoneWaves>(red, row) + down_sum(P, down)) + __half2float(de)) + __half2float(dn));
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

hipError_t launch_lone_dense(NarrowParams P, int grid, hipStream_t s)
{
    P.rows = min(16, (P.dm.h + grid - 1) / grid);
    hipLaunchKernelGGL(k_lone_dense, dim3((P.dm.h + P.rows - 1) / P.rows), dim3(kLoneThreads), lone_dense_lds(), s, P);
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
    return hipFuncSetAttribute((const void *)k_lone_dense, hipFuncAttributeMaxDynamicSharedMemorySize, lone_dense_lds());
}

}  // namespace cfpp
