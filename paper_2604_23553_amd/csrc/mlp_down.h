// MLP-down of the batched path, beside the attention (narrow_attention.hip, group_attention.hip).
#pragma once
#include <type_traits>
#include "decode_params.h"
#include "lone_stream.h"

namespace cfpp {

constexpr int kAttnBatchMax = 8, kAttnBatchThreads = 256;
// What a maximum of scores starts at.  Not minus infinity: the weight of a score of minus infinity (masked, or of an infinite K element) is then
// zero as it comes, with or without others beside it, and so is what no key has been added to.
constexpr float kAttnLowest = -3.402823466e38f;

// MLP-down beside the attention, in workgroups of the same launch behind the attention's: it depends on GELU(up) alone, and an attention
// that is short of bytes, or waits for its merges, leaves the way from memory to these weights.  Workgroup `id` has the rows of
// one group and one part of K, each of its wavefronts a quarter of that, streamed as in narrow_stream.h; the parts are added by
// the output projection, which is a launch of h x h weights alone now.  us per layer of a stack (a block where one is named), both
// products in the launch behind the attention -> this: hidden 2560: five sequences of 37 .. 2048 positions 46.9 -> 44.2, eight
// of 100 .. 300 44.5 -> 39.6, eight prompt tokens behind 1000 46.3 -> 41.7, one block of 1024 positions 37.2 -> 34.1; hidden 4096:
// two of 500 .. 700 78.1 -> 73.7, a block of 1777 positions 76.6 -> 70.9; hidden 1024: eight prompt tokens 21.8 -> 19.7; 1280: two of up
// to 600 23.5 -> 21.5; 512: one sequence, a layer of a stack 15.8 -> 15.2 (a block on its own 14.4, as before).
// Behind the attention's workgroups: ahead of them the block of 1024 positions takes 37.1 us, five sequences the same,
// eight prompt tokens of hidden 4096 5 % more.
struct DownPlan {
    const __half *w;        // packed layer
    int parts, first;       // parts of K; the launch's first workgroup of this kind
};
template <bool ONE>
using DownStream = std::conditional_t<ONE, LoneStream<kDownRowsOne / 16, 4, true>, NgStream<kDownRows / 16, 1, kNgPlanes, 2>>;
template <bool ONE> constexpr int down_lds() { return kAttnBatchThreads / 64 * DownStream<ONE>::kStage; }

template <bool ONE>
__device__ __forceinline__ void mlp_down(const StepParams &P, const DownPlan &plan, int id, int nb, char *lds)
{
    using Stream = DownStream<ONE>;
    constexpr int W = kAttnBatchThreads / 64, ROWS = ONE ? kDownRowsOne : kDownRows;
    const int f = P.dm.f, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = id / plan.parts, z = id - g * plan.parts, r0 = g * ROWS;           // (hidden: a multiple of 128)
    const int C = f / kNgChunk, z0 = C * z / plan.parts, zn = C * (z + 1) / plan.parts - z0, c0 = z0 + zn * wave / W;
    Stream st;
    st.p0.w = plan.w + P.lay.w_down + (size_t)r0 * f; st.p0.row_bytes = (unsigned)f * 2u;
    st.p0.c0 = c0; st.p0.n = z0 + zn * (wave + 1) / W - c0;
    st.ring = lds_address(lds) + (unsigned)(wave * Stream::kStage);
    st.mem = lds + wave * Stream::kStage;
    float *red = reinterpret_cast<float *>(lds), *part = P.part;
    if constexpr (ONE) {
        st.act = P.m; st.act_bytes = (unsigned)f * 4u;
        st.y = nullptr;
        st.begin(ROWS, tid);
        st.run();
        __syncthreads();                                   // the rings have been read
        st.leave(red, wave);
        __syncthreads();
        if (tid < ROWS) part[down_at(0, r0 + tid, z, P.dm.H, P.dm.d, P.part_slots)] = Stream::template total<W>(red, tid);
    } else {
        st.p0.b = P.m; st.p0.b_bytes = (unsigned)nb * (unsigned)f * 4u;
        st.p1 = st.p0; st.p1.n = 0;
        st.gamma = nullptr;
        st.begin(ROWS, nb, nb, 0u, tid);
        st.run();
        __syncthreads();
        st.template leave<1>(red, wave, 0);
        __syncthreads();
        const int row = tid & (ROWS - 1), b = tid / ROWS;  // (256 threads: 8 tokens of 32 rows)
        if (b < nb) part[down_at(b, r0 + row, z, P.dm.H, P.dm.d, P.part_slots)] = ng_total<W>(red, Stream::kSetFloats, row, b);
    }
}

}  // namespace cfpp
