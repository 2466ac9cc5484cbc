// Arguments of the prompt-sized kernels (prefill_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "layout.h"

namespace cfpp {

constexpr int kPfTile = 128;           // hidden, ffn and the scratch's rows are whole multiples of this
constexpr int kPfMaxRows = 4096;       // most tokens a pass takes
// bytes of the parts of a split product: what 384 tiles of 128 x 128 floats take, less the padding of the activation rows
CFPP_HD size_t pf_part_bytes(int rows) { return (size_t)384 * kPfTile * kPfTile * 4 - (size_t)rows * 1024; }

// Halves between the rows of an activation buffer of `width` values a row: 256 bytes more than the
// values take, so that rows at one K offset - what a GEMM step reads - start in different memory channels.
CFPP_HD size_t pf_row_halves(int width) { return 2 * (size_t)width + 128; }

// Scratch of one pass over `rows` tokens (rows a multiple of kPfTile), byte
// offsets; the caller owns the memory.  Activations that feed a GEMM are kept
// as two fp16 planes, head and remainder (half_split.h), interleaved: a row is
// groups of 64 halves, the heads of 32 consecutive values and then their remainders, so that
// 32 values of K are one 128-byte line (see pf_at); rows sit pf_row_halves apart.
struct PfLayout {
    size_t xres, xnext;            // float [rows][h]: residual stream entering / leaving the block
    size_t o;                      // half [rows][2 h + pad]: attention output
    size_t m;                      // half [rows][2 f + pad]: GELU(up)
    size_t stats;                  // float2 [rows]: mean, 1 / sqrt(variance + eps)
    size_t y1, y2;                 // half [rows][2 h + pad]: gamma_1 * x and gamma_2 * x
    size_t q;                      // float [rows][h]: rotated queries
    size_t part;                   // float [parts][rows][columns]: the parts of a product whose K is split over workgroups
    size_t total;                  // (the second product's parts start at q or y1: what lies between is no longer needed then)
};

CFPP_HD PfLayout pf_layout(const Dims &m, int rows)
{
    PfLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    const size_t rh = (size_t)rows * m.h, ah = (size_t)rows * pf_row_halves(m.h) * 2, af = (size_t)rows * pf_row_halves(m.f) * 2;
    L.xres = take(rh * 4); L.xnext = take(rh * 4);
    L.o = take(ah);
    L.m = take(af);
    L.stats = take((size_t)rows * 8);
    L.y1 = take(ah); L.y2 = take(ah);
    L.q = take(rh * 4);
    L.part = take(pf_part_bytes(rows));
    L.total = o;
    return L;
}

// tile (index into the table of prefill_gemm.hip) and splits of K of a product
constexpr int kPfTileKinds = 14;
struct PfPlan { int tile, splits; };

// Passes of up to this many tokens may take the narrow products (prefill_narrow.hip); the activations that feed a
// product are then in their order (ng_at with room for 8 tokens a block) instead of pf_at's.
constexpr int kPfNarrowMax = 64;
struct PfNarrow {
    bool on;
    int rows_in, wgs_q, wgs_in;     // first product: rows of a workgroup, workgroups of the QKV matrix and in all
    // second product: MLP-down beside the attention in `downs` parts of K, the output projection behind it in plan_out.splits - downs,
    // with rows_out rows to a workgroup; downs 0: both behind the attention, as one product over the concatenated K
    int downs, rows_out;
};

// the parts of a split attention (k_pf_attn): unnormalised sums [parts][tokens][h], maximum and weight [parts][tokens][H]
struct PfAttnParts {
    float *o;
    float2 *ml;
    int parts;
    int blocks, first_down; // blocks of queries; the first workgroup that has MLP-down (prefill_beside.hip)
};

struct PfParams {
    Dims dm;
    PackedLayout lay;
    const __half *w;        // packed layer
    const __half *w_next;   // the layer behind it (last layer: unused)
    __half *kv;             // the layer's cache
    int b;                  // sequence inside the cache
    int pos0;               // position of the pass's first token
    int n_rows, rows;       // tokens in this pass, rows of the scratch (n_rows <= rows)
    int layer, n_layers;
    const __half *x_in;     // [n_rows][h] fp16: input of layer 0
    __half *out;            // [n_rows][h] fp16: output of the last layer
    float *xres, *xnext;
    __half *y1, *y2;
    float2 *stats;
    float *q;
    __half *o, *m;
    float *part;            // parts of the first product (QKV, MLP-up), part_bytes
    float *part_out;        // parts of the second one, part_out_bytes
    size_t part_bytes, part_out_bytes, part_out_stride;     // (stride: floats between the second product's parts)
    PfPlan plan_in, plan_out;
    // the first product in two launches (pf_plan_long): MLP-up rows [up_cut, f) with the tile up_tile (up_cut = f: one launch); what a
    // launch takes: the QKV matrix or not, MLP-up rows [up0, up1)
    int up_cut, up_tile;
    int up0, up1;
    bool qkv;
    PfNarrow nrw;
    bool row_fused;         // the kernel that adds the second product's parts prepares the next layer's input too
    const float2 *rope;
};

// where a pass's buffers lie in the scratch at `sc`
inline void pf_place(PfParams &P, const PfLayout &pl, char *sc)
{
    P.y1 = reinterpret_cast<__half *>(sc + pl.y1);
    P.y2 = reinterpret_cast<__half *>(sc + pl.y2);
    P.stats = reinterpret_cast<float2 *>(sc + pl.stats);
    P.q = reinterpret_cast<float *>(sc + pl.q);
    P.o = reinterpret_cast<__half *>(sc + pl.o);
    P.m = reinterpret_cast<__half *>(sc + pl.m);
    P.part = reinterpret_cast<float *>(sc + pl.part); P.part_bytes = pl.total - pl.part;
    P.part_out_bytes = pl.total - pl.q;                    // (where they start: pf_plan_pass)
}

bool pf_supported(const Dims &dm);
// fills in the plans of a pass: everything else of P that does not depend on the layer is set
void pf_plan_pass(PfParams &P);
// behind it, for passes that the narrow products don't take: other tiles for 65 .. 1024 tokens
void pf_plan_middle(PfParams &P);
// behind that, for more than 512 tokens: other tiles for the first product, or two launches
void pf_plan_long(PfParams &P);
// the plan, and what the products' DMA would request past their operands (profiling library): see cfpp_debug_prefill_plan
void pf_describe_plan(const PfParams &P, int plan[8], int past[4]);
void pf_describe_long(const PfParams &P, int plan[5], int past[2]);
// the epilogues' GELU and the library's on n values (profiling library)
hipError_t launch_debug_gelu(const float *z, float *epilogue, float *library, int n, int flags, hipStream_t s);
// one block for the tokens of a pass: LayerNorm inputs, QKV and up, attention, dense and down
hipError_t launch_pf_layer(const PfParams &P, hipStream_t s);
// its products (prefill_gemm.hip): QKV and MLP-up; output projection and MLP-down
hipError_t launch_pf_gemm_in(const PfParams &P, hipStream_t s);
hipError_t launch_pf_gemm_out(const PfParams &P, hipStream_t s);
// The narrow products (prefill_narrow.hip).  pf_plan_narrow: behind pf_plan_pass; true, and P for them, if the pass takes them.
bool pf_plan_narrow(PfParams &P, int n_cu);
// (prefill_beside.hip) the attention with MLP-down in the same launch; parts of K that it takes for so many tokens, 0: it does not
constexpr int kPfDownParts = 8;
hipError_t launch_pf_attention_beside(const PfParams &P, const PfAttnParts &A, hipStream_t s);
int pf_down_parts(const Dims &dm, int tokens);
int pf_down_rows(int tokens);          // rows of a workgroup of MLP-down there
int pf_attn_parts(const PfParams &P);  // parts of the attention's keys (prefill_kernels.hip)
void pf_describe_narrow(const PfParams &P, int plan[7]);   // (profiling library: cfpp_debug_prefill_narrow)
void pf_describe_beside(const PfParams &P, int plan[5]);   // (profiling library: cfpp_debug_prefill_beside)
hipError_t launch_pf_narrow_in(const PfParams &P, hipStream_t s);
hipError_t launch_pf_narrow_out(const PfParams &P, hipStream_t s);

}  // namespace cfpp
