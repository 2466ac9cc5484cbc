// The steps either side of the decode stack in a generation loop (paper Sec.
// 2.3: one graph replay per generated token with static buffers; Sec. 3 compares
// the generated tokens with the baseline's without naming the rule that picks
// them - the largest logit is taken here): the embedding row of the current token before it, and behind it
// the final LayerNorm, the bias-free LM head, and the index of the largest
// logit (lowest index among equal maxima), which becomes the next token while
// the position advances by one.
//
//   k_lm_embed : x[h] = embed[tokens[pos]]
//   k_lm_ring  : LayerNorm, head and pick in one launch (most shapes); the others:
//   k_lm_head  : every workgroup normalises the hidden vector (it is a few KB),
//                streams its share of the LM-head rows like any other GEMV of
//                this library and leaves the best (logit, row) of its share
//   k_lm_pick  : one workgroup picks the best of those in workgroup order,
//                writes tokens[pos + 1] and advances pos
//
// All read pos from device memory and do nothing when it is outside
// [0, max_seq) (the stack kernels raise the error flag for that).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <climits>
#include "decode_blocks.h"
#include "lm_params.h"
#include "lone_stream.h"

namespace cfpp {

__global__ void __launch_bounds__(256) k_lm_embed(LmParams L)
{
    const int p = *L.pos;
    if (p < 0 || p >= L.max_seq) return;
    int tok = L.tokens[p];
    if (tok < 0 || tok >= L.vocab) {
        if (threadIdx.x == 0)
            __hip_atomic_store(&L.sync[kSyncErr], (unsigned)kErrBadToken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tok = 0;
    }
    const u32x4 *src = reinterpret_cast<const u32x4 *>(L.embed + (size_t)tok * L.h);
    u32x4 *dst = reinterpret_cast<u32x4 *>(L.x);
    for (int i = threadIdx.x; i < L.h / 8; i += blockDim.x) dst[i] = src[i];
}

// (logit, row) pairs: a beats b if its logit is larger, or equal with a lower row
__device__ __forceinline__ bool lm_better(float va, int ia, float vb, int ib)
{
    return va > vb || (va == vb && ia < ib);
}

__device__ __forceinline__ void lm_wave_best(float &v, int &i)
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
        const float ov = __shfl_xor(v, m, 64);
        const int oi = __shfl_xor(i, m, 64);
        if (lm_better(ov, oi, v, i)) { v = ov; i = oi; }
    }
}

__global__ void __launch_bounds__(kMaxThreads) k_lm_head(LmParams L)
{
    extern __shared__ __align__(16) float lds[];
    const int p = *L.pos;
    if (p < 0 || p >= L.max_seq) return;
    const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, h = L.h;
    const int Kp = round_up_chunk(h);
    float *y = lds, *part = lds + Kp, *red = part + L.rows * nw;
    const int r_begin = blockIdx.x * L.rows;
    const int r_n = max(0, min(L.rows, L.vocab - r_begin));

    // the first weights are requested before the LayerNorm needs anything
    GemvSpan<kGemvU> gs;
    gs.init(GemvSeg{L.w_lm + (size_t)r_begin * h, y, h, r_n}, GemvSeg{L.w_lm, y, h, 0}, L.w_lm, tid);
    gs.issue_first();
    gs.issue_second();

    // final LayerNorm (two passes, biased variance), output in GEMV order, zero padded
    float xv[kLmPerThread];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < kLmPerThread; ++j) {
        const int i = tid + j * nt;
        xv[j] = i < h ? __half2float(L.hidden[i]) : 0.f;
        s += xv[j];
    }
    const float mean = block_sum(s, red, tid) / (float)h;
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < kLmPerThread; ++j) {
        const float dlt = tid + j * nt < h ? xv[j] - mean : 0.f;
        v += dlt * dlt;
    }
    const float var = block_sum(v, red, tid) / (float)h;
    const float inv = 1.0f / sqrtf(var + L.eps);
#pragma unroll
    for (int j = 0; j < kLmPerThread; ++j) {
        const int i = tid + j * nt;
        if (i < Kp)
            y[lds_perm(i)] = i < h ? (xv[j] - mean) * inv * __half2float(L.lnf_g[i]) + __half2float(L.lnf_b[i]) : 0.f;
    }
    clear_partials(part, L.rows * nw, tid);
    __syncthreads();
    gs.run(part);
    __syncthreads();

    // logits of this workgroup's rows; its best row
    float best = -INFINITY;
    int bi = INT_MAX;
    for (int t = tid; t < r_n; t += nt) {
        const float lg = gs.row_total(part, t);
        if (L.logits) L.logits[r_begin + t] = lg;
        if (lm_better(lg, r_begin + t, best, bi)) { best = lg; bi = r_begin + t; }
    }
    lm_wave_best(best, bi);
    __syncthreads();                                       // red was read by the block sums
    if ((tid & 63) == 0) { red[2 * (tid >> 6)] = best; red[2 * (tid >> 6) + 1] = __int_as_float(bi); }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < nw; ++w) {
            const float ov = red[2 * w];
            const int oi = __float_as_int(red[2 * w + 1]);
            if (lm_better(ov, oi, best, bi)) { best = ov; bi = oi; }
        }
        L.best[2 * blockIdx.x] = best;
        L.best[2 * blockIdx.x + 1] = __int_as_float(bi);
    }
}

__global__ void __launch_bounds__(64) k_lm_pick(LmParams L, int n_wg)
{
    const int p = *L.pos;
    if (p < 0 || p >= L.max_seq) return;
    const int lane = threadIdx.x;
    float best = -INFINITY;
    int bi = INT_MAX;
    for (int g = lane; g < n_wg; g += 64) {
        const float ov = L.best[2 * g];
        const int oi = __float_as_int(L.best[2 * g + 1]);
        if (lm_better(ov, oi, best, bi)) { best = ov; bi = oi; }
    }
    lm_wave_best(best, bi);
    if (lane == 0) {
        L.tokens_out[p + 1] = bi >= 0 && bi < L.vocab ? bi : 0;   // (no finite logit at all: token 0)
        *L.pos_out = p + 1;
    }
}

// The same with the weights through LDS rings (lone_stream.h): hidden sizes in whole chunks of 64 columns, up to 4096, 512 threads.
// A wavefront streams its eighth of the columns of all rows of the workgroup, 16 rows of a chunk at a time, without a break
// between the rows: a row group's sums leave for LDS while the next group's weights are on their way.  The workgroup that delivers the last
// best row picks, in workgroup order: no launch of its own.
// Bound by the weights' way from memory (257 MB of 50304 x 2560: 36.8 us at 7 TB/s).  us of a step of four layers with its head, rows through
// registers and a pick of its own -> this: hidden 512 81.0 -> 77.1, 1280 129.5 -> 109.1, 2560 194.6 -> 183.8; two layers of 4096 217.1 -> 216.4.  Head
// and pick at 2560: 50.3 + 5.3 -> 45.9.  8 or 12 loads in flight: the same.
constexpr int kLmWaves = 8, kLmRing = 8;                   // loads of 1 KiB in flight to a wavefront
constexpr int lm_ring_lds(int rows) { return kLmWaves * (kLmRing * 1024 + kLoneNorm + rows * 4) + 256; }
__global__ void __launch_bounds__(64 * kLmWaves, 2) k_lm_ring(LmParams L)
{
    extern __shared__ __align__(16) char ring_lds[];
    const int h = L.h, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = blockIdx.x * L.rows, rn = max(0, min(L.rows, L.vocab - r0)), groups = (rn + 15) >> 4;
    const int C = h / kNgChunk, c0 = C * wave / kLmWaves, cn = C * (wave + 1) / kLmWaves - c0, n = groups * cn;     // (16 rows of a chunk each)
    char *vec = ring_lds + kLmWaves * kLmRing * 1024, *mine = ring_lds + wave * kLmRing * 1024;
    const int stride = (L.rows + 15) & ~15;
    float *red = reinterpret_cast<float *>(vec + kLmWaves * kLoneNorm);    // [wavefront][row]
    float *last = red + kLmWaves * stride;
    LoneNorm<kLmWaves> norm;
    norm.request(vec, c0, cn, L.hidden, true, L.lnf_g, L.lnf_b, tid);
    const i32x4 rs = dma_rsrc(L.w_lm + (size_t)r0 * h, (unsigned)rn * (unsigned)h * 2u);
    int ig = 0, ic = 0;                                    // what is requested next: group, chunk (past the end: one line over and over)
    auto request = [&](int place) {
        const bool live = ig < groups;
        const unsigned from = (unsigned)__builtin_amdgcn_readfirstlane(live ? (c0 + ic) * 128 : 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int row = min(16 * ig + 8 * k + (lane >> 3), rn - 1);
            lds_dma16_once(rs, lds_address(mine) + (unsigned)(2 * place + k) * 1024u, live ? (unsigned)row * (unsigned)h * 2u + (unsigned)(lane & 7) * 16u : 0u, from);
        }
        if (++ic == cn) { ic = 0; ++ig; }
    };
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < kLmRing / 2; ++i) request(i);
        ng_wait<kLmRing>();                                // x, gamma and beta are there
    } else {
        ng_wait<0>();
    }
    // (ahead of this a vector load would have to wait for the first weights)
    typedef const __attribute__((address_space(4))) int *Scalar;
    const int p = *(Scalar)reinterpret_cast<unsigned long long>(L.pos);
    norm.finish(h, L.eps);
    const float *y = reinterpret_cast<const float *>(vec + wave * kLoneNorm) + (lane & 7) * 8;
    float acc[2] = {0.f, 0.f};
    int g = 0, c = 0;
    for (int i = 0; i < n; i += kLmRing / 2) {
#pragma unroll
        for (int u = 0; u < kLmRing / 2; ++u) {
            if (i + u >= n) break;                         // (uniform)
            ng_wait<kLmRing - 2>();
            const u32x4 w0 = *reinterpret_cast<const u32x4 *>(mine + 2 * u * 1024 + lane * 16), w1 = *reinterpret_cast<const u32x4 *>(mine + (2 * u + 1) * 1024 + lane * 16);
            const float4 *at = reinterpret_cast<const float4 *>(y + c * kNgChunk);
            const float4 ya = at[0], yb = at[1];
            ng_lds_read();                                 // the place in the ring is free
            request(u);
            acc[0] += dot8(w0, ya, yb, 0.f);
            acc[1] += dot8(w1, ya, yb, 0.f);
            if (++c == cn) {                               // (uniform) the group's columns are through
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    float v = acc[k];
                    v += dpp_mov<kDppXor1>(v);
                    v += dpp_mov<kDppXor2>(v);
                    v += dpp_mov<kDppHalfMirror>(v);
                    if ((lane & 7) == 0) red[wave * stride + 16 * g + 8 * k + (lane >> 3)] = v;
                    acc[k] = 0.f;
                }
                c = 0; ++g;
            }
        }
    }
    ng_wait<0>();                                          // (nothing may be on its way to LDS when the workgroup ends)
    __syncthreads();
    if (p < 0 || p >= L.max_seq) return;                   // (uniform over the grid)
    // logits of this workgroup's rows; its best row
    float best = -INFINITY;
    int bi = INT_MAX;
    for (int t = tid; t < rn; t += 64 * kLmWaves) {
        float lg = 0.f;
#pragma unroll
        for (int w = 0; w < kLmWaves; ++w)
            if (C * (w + 1) / kLmWaves > C * w / kLmWaves) lg += red[w * stride + t];
        if (L.logits) L.logits[r0 + t] = lg;
        if (lm_better(lg, r0 + t, best, bi)) { best = lg; bi = r0 + t; }
    }
    lm_wave_best(best, bi);
    if (lane == 0) { last[2 * wave] = best; last[2 * wave + 1] = __int_as_float(bi); }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < kLmWaves; ++w) {
        const float ov = last[2 * w];
        const int oi = __float_as_int(last[2 * w + 1]);
        if (lm_better(ov, oi, best, bi)) { best = ov; bi = oi; }
    }
    unsigned old = 0;
    if (lane == 0) {
        xwg_store(L.best + 2 * blockIdx.x, best);
        xwg_store(L.best + 2 * blockIdx.x + 1, __int_as_float(bi));
        xwg_wait_stores();
        old = __hip_atomic_fetch_add(&L.sync[kSyncLm], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if ((unsigned)__builtin_amdgcn_readfirstlane((int)old) != gridDim.x - 1) return;
    best = -INFINITY;
    bi = INT_MAX;
    for (int w = lane; w < (int)gridDim.x; w += 64) {
        const float ov = xwg_load(L.best + 2 * w);
        const int oi = __float_as_int(xwg_load(L.best + 2 * w + 1));
        if (lm_better(ov, oi, best, bi)) { best = ov; bi = oi; }
    }
    lm_wave_best(best, bi);
    if (lane == 0) {
        L.tokens_out[p + 1] = bi >= 0 && bi < L.vocab ? bi : 0;   // (no finite logit at all: token 0)
        *L.pos_out = p + 1;
        __hip_atomic_store(&L.sync[kSyncLm], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

hipError_t launch_lm_embed(const LmParams &L, hipStream_t s)
{
    hipLaunchKernelGGL(k_lm_embed, dim3(1), dim3(256), 0, s, L);
    return hipGetLastError();
}

size_t lm_head_lds_bytes(const LmParams &L, int threads)
{
    const size_t Kp = (size_t)(L.h + kChunk - 1) / kChunk * kChunk;
    return (Kp + (size_t)L.rows * (threads / 64) + 32) * 4;
}

hipError_t launch_lm_head(const LmParams &L, int grid, int threads, hipStream_t s)
{
    const int ring = lm_ring_lds((L.rows + 15) & ~15);
    if (threads == 64 * kLmWaves && L.h % kNgChunk == 0 && L.h <= 4096 && ring <= 160 * 1024) {
        hipLaunchKernelGGL(k_lm_ring, dim3(grid), dim3(threads), ring, s, L);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_lm_head, dim3(grid), dim3(threads), lm_head_lds_bytes(L, threads), s, L);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lm_pick, dim3(1), dim3(64), 0, s, L, grid);
    return hipGetLastError();
}

hipError_t prepare_lm_kernels(size_t lds_bytes)
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_lm_ring), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(k_lm_head), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds_bytes);
}

}  // namespace cfpp
