// Arguments of the narrow products (narrow_gemm.hip, lone_gemm.hip): a layer's projections for a few tokens - sequences
// of a decode step or a single one, a group of prompt tokens, or a short prompt.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "layout.h"

namespace cfpp {

constexpr int kNgSet = 8;              // tokens whose heads and remainders are the 16 columns of a matrix instruction
constexpr int kBatMax = kNgSet;        // sequences per launch of the batched path

// Activations that feed a narrow product: fp16 heads and remainders in the order in which the matrix instruction
// takes them.  A set of (up to) 8 tokens is K / 32 blocks; a block holds, for each of its four groups of 8 columns, the
// heads of the set's tokens and then their remainders, 8 halves each: one contiguous load of 128 bytes a token.
// nt: tokens a block has room for (8, or those there are, where only one set exists).  The remainder of a value is 8 nt
// halves behind its head.
CFPP_HD size_t ng_at(int token, int k, int width, int nt)
{
    return (size_t)(token >> 3) * width * 16 + (size_t)(k >> 5) * (64 * nt) + ((k >> 3) & 3) * (16 * nt) + (token & 7) * 8 + (k & 7);
}

struct NarrowParams {
    Dims dm;
    PackedLayout lay;
    const __half *w;        // packed layer
    __half *kv;             // the layer's cache
    const int *pos;         // positions of the tokens, device (checked)
    int n, nt;              // tokens; ng_at's nt
    // token i appends to the cache of sequence kv_b0 + i * kv_bstep: its own sequence (first of the group, 1), or -
    // consecutive positions of one prompt - all the same one (b, 0)
    int kv_b0, kv_bstep;
    int layer, n_layers;    // position in the fp32 residual ping-pong
    const __half *x_in;     // [n][h] fp16: input of layer 0
    __half *out;            // [n][h] fp16: output of the last layer
    float *xres;            // [n][2][h]
    float *q;               // [n][h]
    __half *m, *o;          // planes (ng_at): GELU(up), attention output
    float *m32, *o32;       // the same in fp32, in the same memory: a single sequence's (lone_gemm.hip)
    const float2 *rope;
    unsigned *sync;
    float *part;            // the attention's partials (StepParams::part), behind which MLP-down's parts are (down_at)
    int part_slots, downs;  // slots of a head; parts of MLP-down
    int rows, wgs_q;        // matrix rows per workgroup, workgroups of the QKV matrix (set by the launcher)
};

// MLP-down runs beside the attention (mlp_down.h), its K cut into up to kDownParts parts, and leaves their sums where
// the partials of the attention end: the last kDownParts slots of every head, which the attention does not use.  Part z of row
// j for token i of the launch:
constexpr int kDownParts = 8;
CFPP_HD size_t down_at(int i, int j, int z, int H, int d, int part_slots)
{
    const int head = j / d;
    return (((size_t)i * H + head) * part_slots + (part_slots - kDownParts + z)) * (d + 2) + (j - head * d);
}
constexpr int kDownRowsOne = 16, kDownRows = 32;       // rows of a workgroup: one sequence, several
// At most 1024 columns to a part.  For several sequences one workgroup to a CU, or two where that is more than 256 KiB of weights
// to one (a wavefront has 8 KiB of them in flight): us per layer with one / two: hidden 2560 41.7 / 41.9, 2048 32.1 / 32.1, 3072 58.1 / 56.1,
// 4096 77.8 / 73.7; but 288 workgroups take 2 - 3 % more of a layer than 240 (hidden 1536 33.5 / 34.6), 320 6 %.  One
// sequence has no planes to read beside its weights: parts as small as they come (hidden 2560, in three / eight: 35.4 / 34.2).
inline int down_parts_of(int h, int f, bool one)
{
    const int most = min(kDownParts, max(1, f / 1024));
    if (one) return most;
    const int per_cu = (size_t)h * f * 2 > (size_t)256 * 256 * 1024 ? 2 : 1;
    return min(most, max(1, per_cu * 256 * kDownRows / h));
}
// Beside the `attn` workgroups of a prompt group's attention, positions `first` .., whose number the host knows: up to half as many
// workgroups more than CUs take longer than one to each, so as many parts as leave it at that, if these are half as many at least (16 heads of 80
// behind 1500, 144 + 200, stay in between: two parts for five).  us a layer, parts as above -> this: 8 tokens of hidden 1280 (328 workgroups -> 248) behind
// 20 / 400 positions 19.7 -> 19.3 / 21.6 -> 20.3; 2 tokens of 1536 (336 -> 240) 20.3 -> 19.1 / 21.9 -> 20.2.  Two parts are few where the attention is next
// to nothing, so they wait for position 128; behind 20 / 127 / 200 / 400: 2 tokens of 2560 (80) 34.3 -> 34.9 / 35.1 -> 35.0 / 35.4 -> 35.0 / 36.4 -> 35.1, of 2560
// (128) 34.6 -> 34.9 / 35.5 -> 35.0 / 36.3 -> 35.1 / 36.2 -> 35.4, 5 of 2048 (128) 28.1 -> 29.6 / 29.2 -> 29.5 / 29.8 -> 29.6 / 31.4 -> 29.6, 3 of 2048 (64) 27.5 -> 28.6 /
// 28.0 -> 28.7 / 28.0 -> 28.7 / 29.1 -> 28.7, 5 of 1920 26.1 -> 28.0 / 26.9 -> 28.0 / 27.1 -> 28.0 / 28.5 -> 28.1: where they cross lies between 60 and 350.
inline int down_parts_beside(int h, int f, bool one, int attn, int first)
{
    const int parts = down_parts_of(h, f, one), groups = h / kDownRows, room = (256 - attn) / groups;
    const bool between = attn + groups * parts > 256 && attn + groups * parts < 384;
    return !one && between && 2 * room >= parts && (room > 2 || first >= 128) ? room : parts;
}
bool bat_supported(const Dims &dm, int grid, int threads);
// several sequences or tokens (narrow_gemm.hip)
// grid: most workgroups of the first product; the output projection has rows of at most 16 to one and may have twice as many
hipError_t launch_bat_in(NarrowParams P, int grid, hipStream_t s);
hipError_t launch_bat_dense(NarrowParams P, int grid, hipStream_t s);
hipError_t prepare_narrow_kernels();
// one (lone_gemm.hip)
hipError_t launch_lone_in(NarrowParams P, int grid, hipStream_t s);
hipError_t launch_lone_dense(NarrowParams P, int grid, hipStream_t s);
hipError_t prepare_lone_kernels();

}  // namespace cfpp
