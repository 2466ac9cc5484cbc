// Projections of a short prompt, up to 64 tokens (paper Sec. 2.2): what takes time is the weights' way from memory, once
// (narrow_stream.h), and launches.
//
//   k_pf_narrow_in  : QKV rows and MLP-up rows of a layer, whole K per workgroup; the epilogue completes the LayerNorm,
//                     rotates, appends, applies GELU
//   k_pf_narrow_out : output projection and MLP-down as one product over the concatenated K, which is cut over workgroups
//                     (the activations of a whole row of K would be more bytes than its weights); the parts are added
//                     where the next layer's input is made (k_pf_row)
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "narrow_stream.h"
#include "prefill_device.h"

namespace cfpp {

// Wavefronts of a workgroup with T tiles and S sets: as many as leave each a ring of one chunk; four where the sums take
// more than the 256 registers that eight allow a lane.
template <int T, int S>
constexpr int pn_waves() { return T * S >= 40 ? 4 : 160 / (2 * T + 2 * S) > 8 ? 8 : 160 / (2 * T + 2 * S); }
// the rings; at the end, in their place, the sums
template <int T, int S>
constexpr int pn_lds_bytes()
{
    const int ring = NgStream<T, S, kNgPlanes, 1>::kStage, red = S * T * kNgTileFloats * 4;
    return pn_waves<T, S>() * (ring > red ? ring : red);
}

// n / d for 0 <= n < 2^15 and d <= 2^7, inv_d within an ulp of 1 / d: (n + 1/2) / d is at least 1 / 2 d away from a whole
// number, the three roundings less than 2^-22 (n + 1/2) / d.
__device__ __forceinline__ int pn_div(int n, float inv_d) { return (int)(((float)n + 0.5f) * inv_d); }

// What follows the products is dealt in items of two rows of a token over all threads.  With rows dealt to threads and sets
// one after the other it took 0.9 us a set (37 tokens at hidden 2560: 4.5 of 24.3 us), most of them the one wavefront's
// that had the rows past 64.
template <int T, int S>
__global__ void __launch_bounds__((64 * pn_waves<T, S>()), (pn_waves<T, S>() > 4 ? 2 : 1)) k_pf_narrow_in(PfParams P)
{
    using Stream = NgStream<T, S, kNgPlanes, 1>;
    constexpr int W = pn_waves<T, S>(), NT = 64 * W, NI = (8 * T * 8 * S + NT - 1) / NT;   // items of a thread, at most
    static_assert(pn_lds_bytes<T, S>() <= 160 * 1024, "");
    extern __shared__ __align__(16) char pn_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wgs_q = P.nrw.wgs_q, rows = P.nrw.rows_in;
    const bool up = (int)blockIdx.x >= wgs_q;
    const int r0 = ((int)blockIdx.x - (up ? wgs_q : 0)) * rows, rn = min(rows, (up ? f : 3 * h) - r0);   // (even)
    // item i of this thread: token 8 e + b, rows r0 + 2 pr and the next
    const int np = rn >> 1, b = tid & (kNgSet - 1);
    const float inv_np = __builtin_amdgcn_rcpf((float)np);
    auto item = [&](int i, int &e, int &pr) {
        const int n = (tid >> 3) + NT / 8 * i;
        e = pn_div(n, inv_np); pr = n - e * np;
        return 8 * e + b < P.n_rows;
    };
    const float inv_d = __builtin_amdgcn_rcpf((float)dm.d);
    auto place = [&](int pr, int &head, int &part, int &dim) {             // of row pair pr of the QKV matrix
        const int p = r0 + 2 * pr, pd = pn_div(p, inv_d);
        dim = p - pd * dm.d;
        head = pn_div(pd, 1.f / 3.f); part = pd - 3 * head;
    };
    // what it needs of memory: requested ahead of the weights, or, where a lane has no registers for it, behind them
    constexpr bool kAhead = T * S <= 30;
    const float4 *rc = reinterpret_cast<const float4 *>(reinterpret_cast<const float2 *>(P.w + (up ? P.lay.rc_up : P.lay.rc_qkv)) + r0);
    float4 k[NI];                                          // row constants
    float2 mi[NI], cs[NI];                                 // mean and 1/sigma; rotation (QKV)
    auto operands = [&](int i) {
        int e, pr;
        item(i, e, pr);
        const int token = min(8 * e + b, P.n_rows - 1);
        k[i] = rc[pr];
        mi[i] = P.stats[token];
        if (!up) {
            int nh, c, dim;
            place(pr, nh, c, dim);
            cs[i] = P.rope[c < 2 && dim < dm.r ? (unsigned)(P.pos0 + token) * (unsigned)(dm.r >> 1) + (unsigned)(dim >> 1) : 0u];
        }
    };
    if (kAhead) {
#pragma unroll
        for (int i = 0; i < NI; ++i) operands(i);
    }
    Stream st;
    const int C = h / kNgChunk, c0 = C * wave / W;
    st.p0.w = P.w + (up ? P.lay.w_up : P.lay.w_qkv) + (size_t)r0 * h;
    st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.b = up ? P.y2 : P.y1;
    st.p0.set_bytes = (unsigned)h * 32u; st.p0.b_bytes = S * st.p0.set_bytes;
    st.p0.c0 = c0; st.p0.n = C * (wave + 1) / W - c0;
    st.p1 = st.p0; st.p1.n = 0;
    st.ring = lds_address(pn_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = pn_lds + wave * Stream::kStage;
    st.gamma = nullptr;
    st.begin(rn, P.n_rows, kNgSet, 0u, tid);
    st.run();
    float *red = reinterpret_cast<float *>(pn_lds);
    __syncthreads();                                       // the rings have been read
    st.template leave<S>(red, wave, 0);
    __syncthreads();
    __half *kc = P.kv + kv_offset(dm, 0, P.b, 0, 0, 0), *vc = P.kv + kv_offset(dm, 1, P.b, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        int e, pr;
        if (!item(i, e, pr)) continue;
        if (!kAhead) operands(i);
        const int token = 8 * e + b;
        const float2 v = ng_total2<W>(red + e * Stream::kSetFloats, S * Stream::kSetFloats, 2 * pr, b);
        float v0 = (v.x - mi[i].x * k[i].x) * mi[i].y + k[i].y, v1 = (v.y - mi[i].x * k[i].z) * mi[i].y + k[i].w;
        if (up) {
            __half hi[2], lo[2];
            split_half(pf_gelu(v0, dm.flags), hi[0], lo[0]);
            split_half(pf_gelu(v1, dm.flags), hi[1], lo[1]);
            __half *m = P.m + ng_at(token, r0 + 2 * pr, f, kNgSet);
            *reinterpret_cast<unsigned *>(m) = *reinterpret_cast<const unsigned *>(hi);
            *reinterpret_cast<unsigned *>(m + 8 * kNgSet) = *reinterpret_cast<const unsigned *>(lo);
            continue;
        }
        int nh, c, dim;
        place(pr, nh, c, dim);
        int d0 = dim, d1 = dim + 1;
        if (c < 2 && dim < dm.r) {
            const float lo = v0 * cs[i].x - v1 * cs[i].y, hi = v1 * cs[i].x + v0 * cs[i].y;
            v0 = lo; v1 = hi;
            d0 = dim >> 1; d1 = (dim >> 1) + (dm.r >> 1);
        }
        if (c == 0) {
            float *q = P.q + (unsigned)(token * h + nh * dm.d);
            q[d0] = v0; q[d1] = v1;
        } else {
            __half *kv = (c == 1 ? kc : vc) + (size_t)(unsigned)nh * (unsigned)(dm.d * dm.max_seq) + (unsigned)(P.pos0 + token) * 16u;
            kv[(unsigned)(d0 >> 4) * (unsigned)dm.max_seq * 16u + (unsigned)(d0 & 15)] = __float2half_rn(v0);
            kv[(unsigned)(d1 >> 4) * (unsigned)dm.max_seq * 16u + (unsigned)(d1 & 15)] = __float2half_rn(v1);
        }
    }
}

// Workgroup z + splits * g: the z-th part of the concatenated K of rows [g rows, ..); its sums go to part z, [token][h].
// (With as many parts as XCDs a part's activations are in one L2.)
template <int T, int S>
__global__ void __launch_bounds__((64 * pn_waves<T, S>()), (pn_waves<T, S>() > 4 ? 2 : 1)) k_pf_narrow_out(PfParams P)
{
    using Stream = NgStream<T, S, kNgPlanes, 1>;
    constexpr int W = pn_waves<T, S>(), NT = 64 * W, NI = (8 * T * 8 * S + NT - 1) / NT;
    extern __shared__ __align__(16) char pn_lds[];
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int downs = P.nrw.downs, splits = P.plan_out.splits - downs, g = (int)blockIdx.x / splits, z = (int)blockIdx.x - g * splits;
    const int r0 = g * P.nrw.rows_out, rn = min(P.nrw.rows_out, h - r0);
    const int C0 = h / kNgChunk, C = downs > 0 ? C0 : (h + f) / kNgChunk, z0 = C * z / splits, zn = C * (z + 1) / splits - z0;
    const int c0 = z0 + zn * wave / W, c1 = z0 + zn * (wave + 1) / W;
    Stream st;
    st.p0.w = P.w + P.lay.w_dense + (size_t)r0 * h; st.p0.row_bytes = (unsigned)h * 2u;
    st.p0.b = P.o; st.p0.set_bytes = (unsigned)h * 32u; st.p0.b_bytes = S * st.p0.set_bytes;
    st.p0.c0 = min(c0, C0); st.p0.n = max(0, min(c1, C0) - c0);
    st.p1.w = P.w + P.lay.w_down + (size_t)r0 * f; st.p1.row_bytes = (unsigned)f * 2u;
    st.p1.b = P.m; st.p1.set_bytes = (unsigned)f * 32u; st.p1.b_bytes = S * st.p1.set_bytes;
    st.p1.c0 = max(0, c0 - C0); st.p1.n = max(0, c1 - max(c0, C0));
    st.ring = lds_address(pn_lds) + (unsigned)(wave * Stream::kStage);
    st.mem = pn_lds + wave * Stream::kStage;
    st.gamma = nullptr;
    st.begin(rn, P.n_rows, kNgSet, 0u, tid);
    st.run();
    float *red = reinterpret_cast<float *>(pn_lds), *part = P.part_out + (size_t)(downs + z) * P.part_out_stride + r0;
    __syncthreads();                                       // the rings have been read
    st.template leave<S>(red, wave, 0);
    __syncthreads();
    // items of two rows of a token, a token's side by side
    const int np = rn >> 1, items = P.n_rows * np;
    const float inv_np = __builtin_amdgcn_rcpf((float)np);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int n = tid + NT * i, token = pn_div(n, inv_np), pr = n - token * np;
        if (n >= items) break;
        const float2 v = ng_total2<W>(red + (token >> 3) * Stream::kSetFloats, S * Stream::kSetFloats, 2 * pr, token & 7);
        *reinterpret_cast<float2 *>(part + (unsigned)(token * h + 2 * pr)) = v;
    }
}

// ---------------------------------------------------------------------------
constexpr int kPnMostSums = 48;        // tiles x sets of a workgroup, at most (pf_plan_narrow)

template <int T, int S>
static hipError_t pn_launch(const PfParams &P, bool in, hipStream_t s)
{
    if constexpr (T * S > kPnMostSums) return hipErrorInvalidValue;
    else {
    constexpr int lds = pn_lds_bytes<T, S>();
    const void *fn = in ? (const void *)k_pf_narrow_in<T, S> : (const void *)k_pf_narrow_out<T, S>;
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    if (in) {
        hipLaunchKernelGGL((k_pf_narrow_in<T, S>), dim3(P.nrw.wgs_in), dim3(64 * pn_waves<T, S>()), lds, s, P);
    } else {
        const int groups = (P.dm.h + P.nrw.rows_out - 1) / P.nrw.rows_out;
        if ((size_t)P.plan_out.splits * P.part_out_stride * sizeof(float) > P.part_out_bytes) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_pf_narrow_out<T, S>), dim3(groups * (P.plan_out.splits - P.nrw.downs)), dim3(64 * pn_waves<T, S>()), lds, s, P);
    }
    return hipGetLastError();
    }
}
// sets of 8 tokens and tiles of 16 rows as they are built
static int pn_sets_of(int tokens) { const int s = (tokens + 7) / 8; return s == 7 ? 8 : s; }
static int pn_tiles_of(int rows) { const int t = (rows + 15) / 16; return t <= 3 ? t : t <= 5 ? 5 : t <= kNgTileMax ? 8 : 0; }
template <int T>
static hipError_t pn_sets(const PfParams &P, bool in, hipStream_t s)
{
    switch (pn_sets_of(P.n_rows)) {
    case 1: return pn_launch<T, 1>(P, in, s);
    case 2: return pn_launch<T, 2>(P, in, s);
    case 3: return pn_launch<T, 3>(P, in, s);
    case 4: return pn_launch<T, 4>(P, in, s);
    case 5: return pn_launch<T, 5>(P, in, s);
    case 6: return pn_launch<T, 6>(P, in, s);
    case 8: return pn_launch<T, 8>(P, in, s);
    }
    return hipErrorInvalidValue;
}
static hipError_t pn_tiles(const PfParams &P, int rows, bool in, hipStream_t s)
{
    switch (pn_tiles_of(rows)) {
    case 1: return pn_sets<1>(P, in, s);
    case 2: return pn_sets<2>(P, in, s);
    case 3: return pn_sets<3>(P, in, s);
    case 5: return pn_sets<5>(P, in, s);
    case 8: return pn_sets<8>(P, in, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_pf_narrow_in(const PfParams &P, hipStream_t s) { return pn_tiles(P, P.nrw.rows_in, true, s); }
hipError_t launch_pf_narrow_out(const PfParams &P, hipStream_t s) { return pn_tiles(P, P.nrw.rows_out, false, s); }

// Rows and parts of K of the second product: the least estimate, in us, of a workgroup's weights at 27 KB/us, the
// activations it reads from the L2 at 90 KB/us (64 tokens' of 2560 columns: 7 us) and the parts' way to memory and back.
static void pn_plan_out(const PfParams &P, int n_cu, bool dense, int *rows, int *splits)
{
    const int h = P.dm.h, C = (dense ? h : h + P.dm.f) / kNgChunk, tokens = (P.n_rows + 7) / 8 * 8;
    float best = 1e30f;
    for (int sp = 1; sp <= 16 && sp <= C; ++sp) {
        for (int per = 1; per <= 2; ++per) {
            const int groups = per * n_cu / sp;
            if (groups < 1) continue;
            const int r = ((h + groups - 1) / groups + 1) & ~1;
            if (r > 16 * kNgTileMax || pn_tiles_of(r) * pn_sets_of(P.n_rows) > kPnMostSums) continue;
            const float kz = (float)((C + sp - 1) / sp) * kNgChunk;
            const float cost = per * (r * kz * 2.f / 27e3f + tokens * kz * 4.f / 90e3f + 2.f) + 0.15f * sp + (float)sp * P.n_rows * h * 8.f / 4e6f;
            if (cost < best) { best = cost; *rows = r; *splits = sp; }
        }
    }
}

// Which passes take the narrow products: those of up to 64 tokens, as long as a CU's rows of the first product are at most
// 128 (8 tiles) and its sums, tiles x sets, at most 48 (more spill registers: 64 tokens of hidden 4096 133 us a layer against
// 127 with tiles).  us per layer, tiled products -> these: hidden 512, 8 / 40 tokens 24.8 -> 17.4 / 28.5 -> 21.0; hidden 1536,
// 8 / 64 34.3 -> 25.5 / 47.5 -> 40.5; hidden 2560, 8 / 40 / 64 53.5 -> 41.9 / 67.9 -> 56.1 / 72.4 -> 68.7; hidden 4096, 8 / 48
// 109.4 -> 82.8 / 123.6 -> 109.5.  (The tiled ones are left where an MLP is much wider than four times hidden, where the
// device shows fewer CUs, and 49 .. 64 tokens from hidden 2944 on.)
// P is touched only where they are taken.
bool pf_plan_narrow(PfParams &P, int n_cu)
{
    PfNarrow N = P.nrw;
    if (P.n_rows > kPfNarrowMax) return false;
    N.rows_in = ng_in_rows(P.dm, n_cu, &N.wgs_q, &N.wgs_in);
    if (N.rows_in == 0 || pn_tiles_of(N.rows_in) * pn_sets_of(P.n_rows) > kPnMostSums) return false;
    const size_t stride = (size_t)P.n_rows * P.dm.h;
    for (N.downs = pf_down_parts(P.dm, P.n_rows);; N.downs = 0) {
        int splits = 0;
        pn_plan_out(P, n_cu, N.downs > 0, &N.rows_out, &splits);
        // The parts lie from the queries on or, beside an attention that reads these, at the end of the scratch, where the attention may
        // leave parts of its own ahead of them.
        const size_t need = (size_t)(splits + N.downs) * stride * sizeof(float), bytes = (need + 255) / 256 * 256, end = P.part_bytes / 256 * 256;
        const size_t room = N.downs > 0 ? end : P.part_bytes + (size_t)((char *)P.part - (char *)P.q);
        if (splits == 0 || (N.downs > 0 ? bytes : need) > room) {
            if (N.downs > 0) continue;                     // (then behind the attention, if there is room for that)
            return false;
        }
        if (N.downs > 0) P.part_bytes = end - bytes;
        P.part_out = N.downs > 0 ? P.part + P.part_bytes / sizeof(float) : reinterpret_cast<float *>(P.q);
        P.part_out_bytes = N.downs > 0 ? bytes : room;
        P.part_out_stride = stride;
        P.plan_out.splits = splits + N.downs;
        P.row_fused = true;
        N.on = true;
        P.nrw = N;
        return true;
    }
}

#ifdef CFPP_PROFILE
void pf_describe_narrow(const PfParams &P, int plan[7])
{
    plan[0] = 1;
    plan[1] = P.nrw.rows_in; plan[2] = pn_tiles_of(P.nrw.rows_in);
    plan[3] = P.nrw.rows_out; plan[4] = pn_tiles_of(P.nrw.rows_out); plan[5] = P.plan_out.splits - P.nrw.downs;
    plan[6] = pn_sets_of(P.n_rows);
}
void pf_describe_beside(const PfParams &P, int plan[5])
{
    plan[0] = 1;
    plan[1] = P.nrw.downs; plan[2] = P.plan_out.splits - P.nrw.downs;
    plan[3] = pf_attn_parts(P);
    plan[4] = P.nrw.downs * ((P.dm.h + pf_down_rows(P.n_rows) - 1) / pf_down_rows(P.n_rows));
}
#endif

}  // namespace cfpp
