// Single-token decode of one GPT-NeoX block on gfx950, batch 1 per launch.
//
// The block (paper Sec. 2.2; residual form of GPT-NeoX, both branches read x)
// is cut into three phases separated by grid-wide dependencies:
//
//   A  LN1(x), LN2(x) (recomputed by every workgroup, x is a few KB)
//      -> QKV rows (+bias, partial rotary, K/V append, q to workspace)
//      -> MLP-up rows (+bias, exact GELU) -> m
//   B  split-KV attention partials over this workgroup's share of cache rows,
//      last-arriver fixed-order combine per head -> o;  MLP-down rows -> g
//   C  output-projection rows, out = x + (W_d o + b_d) + g
//
// Every matrix is row-split over workgroups (a workgroup owns whole output
// rows), so the only cross-workgroup reduction is the split-KV combine, which
// runs in a fixed order.  Nothing here uses floating-point atomics, so the
// output is bit-identical from run to run (unlike the fp16-atomic output
// accumulation the paper describes in Sec. 3).
//
// The same phase bodies are launched either as three kernels per block or as
// one persistent kernel per block (phases separated by a grid barrier); the
// whole-stack kernel is in fused_kernel.hip.  Sec. 2.3's graph mode wraps any
// of them.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "decode_blocks.h"
#include "attention_blocks.h"
#include "half_split.h"
#include "narrow_params.h"

namespace cfpp {

// ---------------------------------------------------------------------------
// Phase A.  LDS: y1[Kp] y2[Kp] part[(rows_qkv + rows_up) * nw] red[16]
template <class Sync>
__device__ __forceinline__ void phase_a(const StepParams &P, const __half *__restrict__ w, __half *__restrict__ kv,
                                        int layer, int pos, float *lds, Sync &sync)
{
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, d = dm.d, r = dm.r;
    const int tid = opaque_thread_index(), nt = blockDim.x, g = blockIdx.x;
    const int Kp = round_up_chunk(h);
    float *y1 = lds, *y2 = lds + Kp, *part = lds + 2 * Kp;
    float *red = part + (P.rows_qkv + P.rows_up) * (nt >> 6);
    const LayerIO io = layer_io(P, layer);

    // weights first: they depend on nothing, so their loads overlap the wait for x
    const int q_begin = g * P.rows_qkv, q_n = (P.parts & kPartQkv) ? max(0, min(P.rows_qkv, 3 * h - q_begin)) : 0;
    const int u_begin = g * P.rows_up, u_n = (P.parts & kPartUp) ? max(0, min(P.rows_up, f - u_begin)) : 0;
    GemvSpan<kGemvU> gs;
    gs.init(GemvSeg{w + P.lay.w_qkv + (size_t)q_begin * h, y1, h, q_n},
            GemvSeg{w + P.lay.w_up + (size_t)u_begin * h, y2, h, u_n}, w, tid);
    clear_partials(part, (P.rows_qkv + P.rows_up) * (nt >> 6), tid);
    // Epilogue items: the lower half of the wavefronts finishes pairs of QKV
    // rows, the upper half MLP-up rows, items dealt wavefront-major inside a
    // half.  What an item adds (biases, the rotary cos/sin) is requested now: a
    // load issued after the GEMV would cost a full memory round trip with
    // nothing left to hide it.
    const __half *bq = w + P.lay.b_qkv, *bu = w + P.lay.b_up;
    const int hw = nt >> 7, estride = 64 * hw;           // wavefronts per half, items per pass
    const bool up_half = (tid >> 6) >= hw;
    const int item0 = (tid & 63) * hw + ((tid >> 6) - (up_half ? hw : 0));
    float bq0 = 0.f, bq1 = 0.f, bu0 = 0.f;
    float2 cs0 = {1.f, 0.f};
    int rot0 = -1;                                         // pair index of this thread's first item in the rotated part, else -1
    if (!up_half && item0 < q_n / 2) {
        const int p = q_begin + 2 * item0;
        const int i = p % d, c = (p / d) % 3;
        bq0 = __half2float(bq[p]); bq1 = __half2float(bq[p + 1]);
        rot0 = c < 2 && i < r ? i >> 1 : -1;
        if (!Sync::kInputsReady && rot0 >= 0) cs0 = P.rope[(size_t)pos * (r >> 1) + rot0];
    }
    if (up_half && item0 < u_n) bu0 = __half2float(bu[u_begin + item0]);

    Tracer tr;
    tr.init(P, gs.wave, 0);
    tr.mark(1);
    if constexpr (!Sync::kInputsReady) gs.issue_first();   // weights stream while x is waited for
    sync.wait();
    tr.mark(2);

    LnPair ln;
    ln.load(P, w, io, tid);
    if constexpr (Sync::kInputsReady) gs.issue_first();    // x is already on its way: it returns first
    gs.issue_second();
    if constexpr (Sync::kInputsReady) {
        // a launch of its own looks at the position behind its first requests, not before them
        if (!pos_ok(P, pos)) return;
        if (rot0 >= 0) cs0 = P.rope[(size_t)pos * (r >> 1) + rot0];
    }
    ln.finish(P, y1, y2, red, tid);
    __syncthreads();
    tr.mark(3);

    gs.run(part);
    tr.mark(4);
    __syncthreads();
    tr.mark(5);

    if (!up_half) {
        // QKV epilogue: one thread per pair of adjacent packed rows
        for (int pr = item0; pr < q_n / 2; pr += estride) {
            const int p = q_begin + 2 * pr;             // packed row, even
            const int pd = p / d, i = p - pd * d;       // i even
            const int n = pd / 3, c = pd - 3 * n;
            const bool rotary = c < 2 && i < r;         // rotary pair (j, j + r/2)
            float b0 = bq0, b1 = bq1;
            float2 cs = cs0;
            if (pr != item0) {                          // more pairs than threads: tiny grids only
                b0 = __half2float(bq[p]); b1 = __half2float(bq[p + 1]);
                if (rotary) cs = P.rope[(size_t)pos * (r >> 1) + (i >> 1)];
            }
            float v0 = gs.row_total(part, 2 * pr) + b0;
            float v1 = gs.row_total(part, 2 * pr + 1) + b1;
            int d0 = i, d1 = i + 1;
            if (rotary) {
                const int j = i >> 1;
                const float lo = v0 * cs.x - v1 * cs.y;
                const float hi = v1 * cs.x + v0 * cs.y;
                v0 = lo; v1 = hi;
                d0 = j; d1 = j + (r >> 1);
            }
            if (c == 0) {
                xwg_store(P.q + n * d + d0, v0);
                xwg_store(P.q + n * d + d1, v1);
            } else {
                xwg_store_half(kv + kv_offset(dm, c - 1, P.b, n, d0, pos), v0);
                xwg_store_half(kv + kv_offset(dm, c - 1, P.b, n, d1, pos), v1);
            }
        }
    } else {
        for (int t = item0; t < u_n; t += estride) {
            const float b = t == item0 ? bu0 : __half2float(bu[u_begin + t]);
            xwg_store(P.m + u_begin + t, gelu_act(gs.row_total(part, q_n + t) + b, dm.flags));
        }
    }
    tr.mark(6);
    sync.arrive();
}

// ---------------------------------------------------------------------------
// A head of few rows is one workgroup's: its output needs no partial, acknowledgement, counter and
// second reading (three dependent trips to memory).  Few: what 8 wavefronts take in four rows each,
// less where the workgroup's own MLP-down rows are long beside it.  us per block, equal shares ->
// whole heads: hidden 512: 128 positions 22.6 -> 21.1, 500: 24.3 -> 23.0, 1000 (32 rows): 28.0 -> 25.3,
// 2000: 28.1 -> 29.6; hidden 1024, 500 (32 rows): 30.8 -> 28.1; hidden 1280, 128: 35.0 -> 33.9, 1000:
// 38.4 -> 38.7; hidden 2560, 300: 43.6 -> 44.3, 1000: 44.6 -> 49.4.  Those rows are the longer the fewer
// workgroups there are; with 64 of them: hidden 512, 450 (15 rows): 24.2 -> 22.4, 1000: 24.3 -> 24.5; hidden
// 1024, 100 (7 rows): 30.9 -> 30.8, 450 (29): 31.8 -> 34.5; with 32: hidden 512, 450: 28.4 -> 28.7, 1000: 28.9 -> 31.4.
// Four wavefronts to a workgroup: hidden 1024, 450: 29.6 -> 27.0, hidden 1280, 780 (25 rows): 41.6 -> 42.5.
__device__ __forceinline__ bool whole_heads(const Dims &dm, int rows, int grid, int nw)
{
    return grid >= dm.H && dm.h < 2048 && rows <= 32 && rows * dm.h <= (nw >= 8 ? 128 : 120) * min(grid, 256);
}

// Split-KV decode attention over this workgroup's share of the cache, all
// wavefronts taking rows round-robin.
// scr: nw*(D+2) + 4 + 2*D floats of LDS.
// pre(): called once, after the first row of already-cached K/V has been
// requested and before anything written during this launch (q, the new token's
// K/V) is read.  early(): called once, when every K/V load of the first two rows
// has been requested (the caller requests what it wants in flight during the
// arithmetic).  mid(): called once, ahead of the first workgroup barrier (the
// caller finishes staging its LDS vectors there).  tail(): called once, when the
// last K/V rows have been consumed, ahead of the last merges.
template <int D, class Pre, class Early, class Mid, class Tail>
__device__ __forceinline__ void attn_share(const StepParams &P, const __half *__restrict__ kv, int n_tok,
                                           float *scr, int tid, Pre &&pre, Early &&early, Mid &&mid, Tail &&tail,
                                           Tracer &tr)
{
    using AC = AttnCore<D>;
    constexpr int NP = AC::NP;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    float *wp = scr, *wm = scr + nw * D, *wl = wm + nw;
    float *qs = wl + nw + 4;                               // this head's query
    __half *kn = reinterpret_cast<__half *>(qs + D);       // the new token's K and V rows of this head
    __half *vn = kn + D;
    AC ac;
    ac.init(P, kv, n_tok, lane);
    const bool whole = whole_heads(P.dm, ac.R, (int)gridDim.x, nw);     // (uniform over the grid)
    if (whole) ac.take_whole_heads();

    if (ac.r0 >= ac.r1 || !(P.parts & kPartAttention)) {   // no rows for this workgroup, or no attention in this launch
        pre();
        early();
        mid();
        __syncthreads();
        tail();
        return;
    }

    // Order of the requests: first row of cached K/V (needs nothing), then -
    // behind the caller's wait - the small vectors written during this launch,
    // then the second row and the caller's next weights.  The small loads return
    // while the bulk behind them is still streaming.
    u32x4 kA[NP], vA[NP], kB[NP], vB[NP];
    HeadStage<D> hst;
    bool first = true;
    {
        int s, se, row_lo, row_hi;
        ac.segment(ac.r0, s, se, row_lo, row_hi);
        const int row = row_lo + wave;
        ac.issue(kA, vA, s, row < row_hi ? row : -1);
        pre();
        hst.issue(P, kv, s, n_tok, tid);
        ac.issue(kB, vB, s, row + nw < row_hi ? row + nw : -1);
        early();
        hst.commit(qs, kn, vn, tid);
        mid();
    }

    for (int sb = ac.r0; sb < ac.r1;) {
        int s, se, row_lo, row_hi;
        ac.segment(sb, s, se, row_lo, row_hi);
        int row = row_lo + wave;
        if (!first) {
            ac.issue(kA, vA, s, row < row_hi ? row : -1);
            hst.issue(P, kv, s, n_tok, tid);
            ac.issue(kB, vB, s, row + nw < row_hi ? row + nw : -1);
            hst.commit(qs, kn, vn, tid);
        }
        first = false;
        __syncthreads();
        ac.reset();
        const bool last_seg = se == ac.r1;
        // Two rows are in flight per wavefront; a register set is refilled as soon
        // as its row is consumed.  The sets swap roles instead of being copied: a
        // copy of a set whose loads are still in flight would have to wait for them.
        // (no exit between the two halves: with one, the load counter's model loses track of
        // which set is older and every wait drains the queue)
        while (row < row_hi) {
            ac.process(kA, vA, row, qs, kn, vn);
            ac.issue(kA, vA, s, row + 2 * nw < row_hi ? row + 2 * nw : -1);
            if (row + nw < row_hi) ac.process(kB, vB, row + nw, qs, kn, vn);
            ac.issue(kB, vB, s, row + 3 * nw < row_hi ? row + 3 * nw : -1);
            row += 2 * nw;
        }

        // The first wavefront alone merges the wavefronts' states, publishes the
        // workgroup's partial and, if it was the last of the head, combines the head;
        // the others go on after one barrier.
        if (last_seg && wave != 0) tail();
        ac.wave_merge(wp, wm, wl, wave);
        tr.mark(14);
        __syncthreads();
        if (wave == 0 && whole) {
            ac.finish(P, s, wp, wm, wl, nw);
            if (last_seg) tail();
        } else if (wave == 0) {
            ac.publish(P, s, wp, wm, wl, nw);
            if (!CFPP_SKIPPED(P, 8)) {
                xwg_wait_stores();
                tr.mark(15);
                if (last_seg) tail();
                ac.count_and_combine(P, s);
            } else if (last_seg) {
                tail();
            }
        }
        if (!last_seg) __syncthreads();                    // the scratch is reused by the next head
        tr.mark(16);
        sb = se;
    }
}

// Phase B.  LDS: m[Kp_f] part[rows_h*nw] scr[nw*(D+2)+4+2*D]
template <int D, class Sync>
__device__ __forceinline__ void phase_b(const StepParams &P, const __half *__restrict__ w,
                                        const __half *__restrict__ kv, int pos, float *lds, Sync &sync)
{
    const Dims &dm = P.dm;
    const int h = dm.h, f = dm.f, tid = opaque_thread_index(), nt = blockDim.x, g = blockIdx.x;
    const int Kp = round_up_chunk(f);
    float *ml = lds, *part = lds + Kp;
    float *scr = part + P.rows_h * (nt >> 6);
    const int r_begin = g * P.rows_h, r_n = (P.parts & kPartDown) ? max(0, min(P.rows_h, h - r_begin)) : 0;
    GemvSpan<kGemvUDown> gs;
    gs.init(GemvSeg{w + P.lay.w_down + (size_t)r_begin * f, ml, f, r_n}, GemvSeg{w + P.lay.w_down, ml, f, 0}, w, tid, kShare0AfterAttention);
    // the first down-projection weights are requested behind the last K/V loads,
    // so that they stream while the attention partials are merged
    Tracer tr;
    tr.init(P, gs.wave, 16);
    tr.mark(10);
    clear_partials(part, P.rows_h * (nt >> 6), tid);
    const __half *bd = w + P.lay.b_down;
    const int item0 = spread_index(tid);
    const float bd0 = item0 < r_n ? __half2float(bd[r_begin + item0]) : 0.f;   // for the epilogue
    StagedVector<kStageM> sm;
    if constexpr (Sync::kInputsReady) sm.issue(P.m, f, tid);
    attn_share<D>(P, kv, pos + 1, scr, tid,
                  [&] {
                      sync.wait();
                      tr.mark(11);
                      if constexpr (!Sync::kInputsReady) sm.issue(P.m, f, tid);
                  },
                  [&] {
                      // The first down-projection weights are requested here, behind the
                      // K/V rows: they stream while the rows are processed and the partials
                      // merged.  (The first wavefront has no share of the GEMV: its loads
                      // re-read one cached block and cost nothing to wait for.)
                      gs.issue_first();
                      gs.issue_second();
                  },
                  [&] { sm.commit(f, ml, tid); tr.mark(12); },
                  [&] { tr.mark(13); }, tr);
    tr.mark(17);
    gs.run(part);            // (m became visible at the barrier inside attn_share)
    tr.mark(18);
    __syncthreads();
    for (int t = item0; t < r_n; t += nt)
        xwg_store(P.g + r_begin + t, gs.row_total(part, t) + (t == item0 ? bd0 : __half2float(bd[r_begin + t])));
    tr.mark(19);
    sync.arrive();
}

// Phase C.  LDS: o[Kp_h] part[rows_h*nw]
template <class Sync>
__device__ __forceinline__ void phase_c(const StepParams &P, const __half *__restrict__ w, int layer,
                                        float *lds, Sync &sync)
{
    const Dims &dm = P.dm;
    const int h = dm.h, tid = opaque_thread_index(), nt = blockDim.x, g = blockIdx.x;
    const int Kp = round_up_chunk(h);
    float *ol = lds, *part = lds + Kp;
    const LayerIO io = layer_io(P, layer);
    const int r_begin = g * P.rows_h, r_n = max(0, min(P.rows_h, h - r_begin));
    const bool dense = P.parts & kPartDense, down = P.parts & kPartDown;   // branches this launch adds to the residual
    GemvSpan<kGemvU> gs;
    gs.init(GemvSeg{w + P.lay.w_dense + (size_t)r_begin * h, ol, h, dense ? r_n : 0}, GemvSeg{w + P.lay.w_dense, ol, h, 0}, w, tid);
    Tracer tr;
    tr.init(P, gs.wave, 48);
    tr.mark(20);
    clear_partials(part, P.rows_h * (nt >> 6), tid);
    StagedVector<kStageM> so;
    if constexpr (Sync::kInputsReady) so.issue(P.o, h, tid);
    gs.issue_first();
    gs.issue_second();
    if constexpr (Sync::kInputsReady) {
        int pos;
        if (!read_pos(P, &pos)) return;
    }
    sync.wait();
    tr.mark(21);
    if constexpr (!Sync::kInputsReady) so.issue(P.o, h, tid);
    // epilogue operands of this thread's first row
    const __half *bd = w + P.lay.b_dense;
    const int item0 = spread_index(tid);
    float bd0 = 0.f, x0 = 0.f, g0 = 0.f;
    if (item0 < r_n) {
        bd0 = __half2float(bd[r_begin + item0]);
        x0 = load_x(io, r_begin + item0);
        g0 = down ? xwg_load(P.g + r_begin + item0) : 0.f;
    }
    so.commit(h, ol, tid);
    __syncthreads();
    tr.mark(22);
    gs.run(part);
    tr.mark(23);
    __syncthreads();
    for (int t = item0; t < r_n; t += nt) {
        const bool pre = t == item0;
        const float a = dense ? gs.row_total(part, t) + (pre ? bd0 : __half2float(bd[r_begin + t])) : 0.f;
        const float res = ((pre ? x0 : load_x(io, r_begin + t)) + a) + (pre ? g0 : (down ? xwg_load(P.g + r_begin + t) : 0.f));
        if (io.o16) io.o16[r_begin + t] = __float2half_rn(res);
        else xwg_store(io.o32 + r_begin + t, res);
    }
    tr.mark(24);
    sync.arrive();
}

// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kMaxThreads)
k_phase_a(StepParams P, const __half *w, __half *kv, int layer)
{
    extern __shared__ __align__(16) float lds[];
    NoSync sync;
    phase_a(P, w, kv, layer, *P.pos, lds, sync);           // (checks the position itself)
}

template <int D>
__global__ void __launch_bounds__(kMaxThreads)
k_phase_b(StepParams P, const __half *w, const __half *kv)
{
    extern __shared__ __align__(16) float lds[];
    int pos;
    if (!read_pos(P, &pos)) return;
    NoSync sync;
    phase_b<D>(P, w, kv, pos, lds, sync);
}

__global__ void __launch_bounds__(kMaxThreads)
k_phase_c(StepParams P, const __half *w, int layer)
{
    extern __shared__ __align__(16) float lds[];
    NoSync sync;
    phase_c(P, w, layer, lds, sync);                       // (checks the position itself)
}

// The attention of several sequences in one launch.  P holds the parameters of the first
// sequence; sequence i follows at the workspace's usual strides.  A workgroup (4 wavefronts,
// several to a CU) takes one piece of ONE head of one sequence: every head of sequence i is cut
// into 1 + spare * rows_i / rows_all pieces, worked out by every workgroup from the positions in
// device memory (the grid is the most that can come out; what is over leaves at once).  So a
// short sequence is as many workgroups as it has heads, and none does several heads one after
// the other: dealing 256 workgroups of 512 threads to the sequences by length left the heads of
// a short one to one or two of them, a staging, merge and hand-over (about 1.2 us) per head.
// Wavefronts interleave the piece's rows (PPW positions each), two rows in flight; the running
// softmax is per lane group and merged lane -> wavefront -> workgroup -> head, each in a fixed
// order; the workgroup that delivers a head's last piece adds the pieces in order.  The new token's
// K and V row is read from the cache like the others (the launch before this one wrote it).
// STREAM: non-temporal loads (every row is read once); without: a group of prompt tokens, whose
// queries read the same rows (attn_bstep = 0).
constexpr int kAttnBatchMax = 8, kAttnBatchThreads = 256;
// Workgroups dealt beyond one per head and sequence, and the fewest rows worth a piece.  us per step and layer, before
// -> with pieces of 8 / 16 / 32 rows: five sequences of 37 .. 2048 positions (hidden 2560) 85.0 -> 65.9 / 65.7 / 63.6;
// 8 prompt tokens behind 1000: 67.3 -> 70.5 / 66.4 / 64.2; two sequences of 8000: 80.0 -> 81.8 / 79.4 / 78.9. 
// Spare ones of sequences with K/V rows of their own: 640, shared out by rows and rounded down per sequence, so that with one
// per head it comes to 650 .. 900 workgroups of about one size for up to 32 heads, about what is resident at 3 a CU.  Chosen at 32 heads and 8
// sequences: one block of hidden 4096, 3219 .. 7696 positions, 256 / 512 / 640 / 1024 / 2048 spare ones: 224.4 / 219.4 /
// 218.2 / 222.7 / 223.7 us (218.2 with the 256 workgroups of before); of 1024 .. 8192 positions 640 / 1024 / 2048: 231.8 /
// 232.0 / 230.4 (234 .. 236 before).  Elsewhere 640 was held against the kernels of before only, us per whole step: 8 heads, 4 layers,
// 2 sequences of 6000 .. 8000 183 -> 157, 8 of 2000 190 -> 169; 24 heads, 4 layers 245 -> 232, 266 -> 257; 32 heads of 80,
// 2 layers 168 -> 156, 182 -> 178.  A prompt group's queries share their
// rows and don't stream: 1024, as measured above.  Pieces of a head never exceed the workspace's part_slots.
constexpr int kAttnSpareGroups = 640, kAttnSpareShared = 1024, kAttnPieceRows = 32;
// Up to four sequences of their own leave workgroups to spare: up to eight pieces of half as many rows.  us a block, 32 rows -> 16:
// hidden 2560, one sequence of 1000 / 2000 / 4000 41.3 -> 39.5 / 43.4 -> 41.0 / 45.4 -> 43.7, three of 500 .. 1000 42.9 -> 41.8;
// hidden 4096, four of 20 .. 2000 85.7 -> 83.6; but five of 37 .. 2048 45.6 -> 47.4, prompt groups 47.0 -> 47.9, and 16 pieces
// of one sequence of 8000 49.7 -> 50.4.
constexpr int kAttnFew = 4;
CFPP_HD int attn_pieces(int rows, bool few)
{
    const int n = (rows + kAttnPieceRows - 1) / kAttnPieceRows, half = (rows + kAttnPieceRows / 2 - 1) / (kAttnPieceRows / 2);
    return !few || n >= 8 ? n : half < 8 ? half : 8;
}

template <int D, bool STREAM, bool ONE>
__global__ void __launch_bounds__(kAttnBatchThreads, 3)
k_attention_batched(StepParams P, int nb, int spare, bool few, const __half *kv)
{
    using A = AttnShape<D>;
    constexpr int LPP = A::LPP, PPW = A::PPW, NP = A::NP, NV = A::NV, NE = (D + 63) / 64, NW = kAttnBatchThreads / 64;
    __shared__ __align__(16) float qs[D];
    __shared__ float wp[NW * D], wm[NW], wl[NW];
    const Dims &dm = P.dm;
    const int H = dm.H, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this workgroup's sequence, head and piece (rows: per head, every head of a sequence has the same number).  All of it
    // stands in front of the first load, so: scalar loads, and reciprocals instead of divisions.
    typedef const __attribute__((address_space(4))) int *Scalar;
    const Scalar positions = (Scalar)reinterpret_cast<unsigned long long>(P.pos);
    int rows[kAttnBatchMax], at[kAttnBatchMax], total = 0;
    bool ok = true;
#pragma unroll
    for (int i = 0; i < kAttnBatchMax; ++i) {
        at[i] = positions[min(i, nb - 1)];
        ok = ok && at[i] >= 0 && at[i] < dm.max_seq;
        rows[i] = i < nb ? (at[i] + 1 + PPW - 1) / PPW : 0;
        total += rows[i];
    }
    if (!ok) {
        if (tid == 0 && blockIdx.x == 0)
            __hip_atomic_store(&P.sync[kSyncErr], (unsigned)kErrBadPos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const float share = (float)spare * __builtin_amdgcn_rcpf((float)total);          // (whatever it is rounded to: the shares' whole parts add up to spare at most)
    int mine = -1, R = 0, pieces = 1, local = 0, base = 0, t_last = 0;
#pragma unroll
    for (int i = 0; i < kAttnBatchMax; ++i) {
        if (i < nb) {
            const int n = min(min(1 + (int)((float)rows[i] * share), attn_pieces(rows[i], few)), P.part_slots);
            const int in = (int)blockIdx.x - base;
            if (in >= 0 && in < n * H) { mine = i; R = rows[i]; pieces = n; local = in; t_last = at[i]; }
            base += n * H;
        }
    }
    if (mine < 0) return;                                  // (whole workgroup)
    // local / H (both below 2^15: the half keeps every quotient off a whole number), and the piece's rows: R / pieces each,
    // the first ones one more
    const int piece = (int)(((float)local + 0.5f) * __builtin_amdgcn_rcpf((float)H)), head = local - piece * H;
    int each = (int)((float)R * __builtin_amdgcn_rcpf((float)pieces)), rest = R - each * pieces;
    if (rest < 0) { --each; rest += pieces; }
    if (rest >= pieces) { ++each; rest -= pieces; }
    const int b = P.b + mine * P.attn_bstep;
    const int lo = piece * each + min(piece, rest), hi = lo + each + (piece < rest);
    const int sub = lane & (LPP - 1), tl = lane / LPP;
    const __half *Kh = kv + kv_offset(dm, 0, b, head, 0, 0), *Vh = kv + kv_offset(dm, 1, b, head, 0, 0);
    unsigned koff[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int pc = sub + LPP * k;
        koff[k] = ((unsigned)(pc >> 1) * (unsigned)dm.max_seq * 16u + (unsigned)(pc & 1) * 8u) * 2u;
    }
    u32x4 k0[NP], v0[NP], k1[NP], v1[NP];
    // always 2 NP loads, every lane active: the load counter tells rows in flight apart (rows past the piece's end
    // and positions past the last re-read the last position; their weight is zero)
    auto issue = [&](u32x4 (&kk)[NP], u32x4 (&vv)[NP], int row) {
        const int t = row < hi ? row * PPW + tl : t_last;
        const unsigned tb = (unsigned)min(t, t_last) * 32u;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            if (STREAM) kk[k] = load16_stream_at(Kh, koff[k] + tb);
            else kk[k] = *as_global(reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(Kh) + (koff[k] + tb)));
        }
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            if (STREAM) vv[k] = load16_stream_at(Vh, koff[k] + tb);
            else vv[k] = *as_global(reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(Vh) + (koff[k] + tb)));
        }
        __builtin_amdgcn_sched_barrier(0);                 // the loads stay here, ahead of the arithmetic
    };
    const float q_r = tid < D ? P.q[(size_t)mine * dm.h + head * D + tid] : 0.f;
    issue(k0, v0, lo + wave);
    issue(k1, v1, lo + wave + NW);
    if (tid < D) qs[tid] = q_r * (1.44269504088896340736f / sqrtf((float)D));
    __syncthreads();
    float acc[NV], m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.f;
    auto process = [&](const u32x4 (&kk)[NP], u32x4 (&vv)[NP], int row) {
        const bool valid = row * PPW + tl <= t_last;
        if (row * PPW + PPW - 1 > t_last) {                // (uniform) a head's last row: the re-read V weighs nothing, infinite or not
#pragma unroll
            for (int k = 0; k < NP; ++k) vv[k] = valid ? vv[k] : u32x4{0u, 0u, 0u, 0u};
        }
        int qoff = 8 * sub;
        asm volatile("" : "+v"(qoff));                     // (q is re-read from LDS for every row, not kept in 8 NP registers)
        float sp = 0.f;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const float4 qa = *reinterpret_cast<const float4 *>(qs + qoff + 8 * LPP * k);
            const float4 qb = *reinterpret_cast<const float4 *>(qs + qoff + 8 * LPP * k + 4);
            sp = dot8(kk[k], qa, qb, sp);
        }
        sp += lane_xor<1>(sp);                             // the lanes sharing this position
        if constexpr (LPP == 4) sp += lane_xor<2>(sp);
        const float sc = valid ? sp : -INFINITY;
        const float mn = fmaxf(m_run, sc);
        const float corr = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mn);
        const float p = valid ? __builtin_amdgcn_exp2f(sc - mn) : 0.f;
        l_run = l_run * corr + p;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const float2 a = unpack_h2(vv[k].x), b2 = unpack_h2(vv[k].y), c = unpack_h2(vv[k].z), e = unpack_h2(vv[k].w);
            float *ac = acc + 8 * k;
            ac[0] = fmaf(p, a.x, ac[0] * corr); ac[1] = fmaf(p, a.y, ac[1] * corr);
            ac[2] = fmaf(p, b2.x, ac[2] * corr); ac[3] = fmaf(p, b2.y, ac[3] * corr);
            ac[4] = fmaf(p, c.x, ac[4] * corr); ac[5] = fmaf(p, c.y, ac[5] * corr);
            ac[6] = fmaf(p, e.x, ac[6] * corr); ac[7] = fmaf(p, e.y, ac[7] * corr);
        }
        m_run = mn;
    };
    for (int r = lo + wave; r < hi; r += 2 * NW) {
        process(k0, v0, r);
        issue(k0, v0, r + 2 * NW);
        if (r + NW < hi) process(k1, v1, r + NW);          // (uniform)
        issue(k1, v1, r + 3 * NW);
    }
    // lanes -> wavefront (a wavefront without rows leaves (0, -inf, 0)) -> workgroup
    {
        const float mw = wave_max(m_run);
        const float fl = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - mw);
        const float lw = wave_sum(sub == 0 ? l_run * fl : 0.f);
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] *= fl;
        int off, cnt;
        reduce_scatter<NV, LPP>(acc, lane, off, cnt);
#pragma unroll
        for (int i = 0; i < A::NLEFT; ++i) {
            if (i < cnt) {
                const int idx = off + i;                   // accumulator index: piece idx / 8, element idx % 8
                wp[wave * D + 8 * (sub + LPP * (idx >> 3)) + (idx & 7)] = acc[i];
            }
        }
        if (lane == 0) { wm[wave] = mw; wl[wave] = lw; }
    }
    __syncthreads();
    if (wave != 0) return;
    float M = wm[0], L = 0.f, O[NE];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, wm[w]);      // (the piece has rows: finite)
#pragma unroll
    for (int e = 0; e < NE; ++e) O[e] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float ew = wm[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wm[w] - M);
        L += wl[w] * ew;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (lane + 64 * e < D) O[e] += wp[w * D + lane + 64 * e] * ew;
    }
    auto deliver = [&]() {                                 // as the output projection takes them: heads and remainders; one sequence's in fp32
        __half *out = reinterpret_cast<__half *>(P.o);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            if (lane + 64 * e >= D) continue;
            if (ONE) { P.o[head * D + lane + 64 * e] = O[e] / L; continue; }
            __half hi, lo;
            split_half(O[e] / L, hi, lo);
            const size_t at = ng_at(mine, head * D + lane + 64 * e, dm.h, nb);
            out[at] = hi; out[at + 8 * nb] = lo;
        }
    };
    if (pieces == 1) {
        deliver();
        return;
    }
    // publish the piece; the last one of the head adds them in order
    const size_t hd = (size_t)mine * H + head;
    float *first = P.part + hd * P.part_slots * (D + 2), *slot = first + (size_t)piece * (D + 2);
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if (lane + 64 * e < D) xwg_store(slot + lane + 64 * e, O[e]);
    if (lane == 0) { xwg_store(slot + D, M); xwg_store(slot + D + 1, L); }
    xwg_wait_stores();
    unsigned old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(&P.seg_cnt[hd], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane((int)old) != pieces - 1) return;
    constexpr int CB = 8;                                  // pieces whose loads are in flight together
    M = -INFINITY; L = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) O[e] = 0.f;
    for (int j0 = 0; j0 < pieces; j0 += CB) {
        float mj[CB], lj[CB], oj[CB][NE];
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const float *sj = first + (size_t)min(j0 + j, pieces - 1) * (D + 2);
            mj[j] = xwg_load(sj + D);
            lj[j] = xwg_load(sj + D + 1);
#pragma unroll
            for (int e = 0; e < NE; ++e) oj[j][e] = xwg_load(sj + (lane + 64 * e < D ? lane + 64 * e : 0));
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            if (j0 + j < pieces) {
                const float mn = fmaxf(M, mj[j]);
                const float c0 = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - mn), c1 = __builtin_amdgcn_exp2f(mj[j] - mn);
                L = L * c0 + lj[j] * c1;
#pragma unroll
                for (int e = 0; e < NE; ++e) O[e] = O[e] * c0 + oj[j][e] * c1;
                M = mn;
            }
        }
    }
    deliver();
    if (lane == 0) __hip_atomic_store(&P.seg_cnt[hd], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int D>
__global__ void __launch_bounds__(kMaxThreads)
k_block_persistent(StepParams P, const __half *w, __half *kv, int layer)
{
    extern __shared__ __align__(16) float lds[];
    int pos;
    if (!read_pos(P, &pos)) return;
    GridBarrier bar;
    bar.init(P.sync, gridDim.x);
    GridSync sync{bar};
    phase_a(P, w, kv, layer, pos, lds, sync);
    phase_b<D>(P, w, kv, pos, lds, sync);
    phase_c(P, w, layer, lds, sync);
    bar.finish();
}

// ---------------------------------------------------------------------------
// host-side launchers

#define CFPP_TRY(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) return e_; } while (0)

template <int D>
static hipError_t launch_phases_d(const StepParams &P, const __half *w, __half *kv, int layer,
                                  int grid, int threads, hipStream_t s)
{
    const size_t lds = (size_t)P.lds_floats * 4;
    hipLaunchKernelGGL(k_phase_a, dim3(grid), dim3(threads), lds, s, P, w, kv, layer);
    CFPP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_phase_b<D>, dim3(grid), dim3(threads), lds, s, P, w, (const __half *)kv);
    CFPP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_phase_c, dim3(grid), dim3(threads), lds, s, P, w, layer);
    return hipGetLastError();
}

hipError_t launch_phases(const StepParams &P, const __half *w, __half *kv, int layer,
                         int grid, int threads, hipStream_t s)
{
    switch (P.dm.d) {
    case 64: return launch_phases_d<64>(P, w, kv, layer, grid, threads, s);
    case 80: return launch_phases_d<80>(P, w, kv, layer, grid, threads, s);
    case 128: return launch_phases_d<128>(P, w, kv, layer, grid, threads, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_attention_batched(const StepParams &P, int nb, const __half *kv, hipStream_t s)
{
    if (nb < 1 || nb > kAttnBatchMax) return hipErrorInvalidValue;
    const bool stream = P.attn_bstep != 0;
    const int H = P.dm.H, spare = (stream ? kAttnSpareGroups : kAttnSpareShared) / H;
    const bool few = stream && nb <= kAttnFew;
    // no sequence has more pieces than its longest context allows (64 / LPP positions a row, as in AttnShape)
    const int row = P.dm.d >= 128 ? 16 : 32, most = attn_pieces((P.dm.max_seq + row - 1) / row, few);
    const dim3 grid(min(nb + spare, nb * most) * H), block(kAttnBatchThreads);
    switch (P.dm.d) {
#define CFPP_ATTN(D) \
    case D: \
        if (stream && nb == 1) hipLaunchKernelGGL((k_attention_batched<D, true, true>), grid, block, 0, s, P, nb, spare, few, kv); \
        else if (stream) hipLaunchKernelGGL((k_attention_batched<D, true, false>), grid, block, 0, s, P, nb, spare, few, kv); \
        else if (nb == 1) hipLaunchKernelGGL((k_attention_batched<D, false, true>), grid, block, 0, s, P, nb, spare, few, kv); \
        else hipLaunchKernelGGL((k_attention_batched<D, false, false>), grid, block, 0, s, P, nb, spare, few, kv); \
        break;
    CFPP_ATTN(64)
    CFPP_ATTN(80)
    CFPP_ATTN(128)
#undef CFPP_ATTN
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_block_persistent(const StepParams &P, const __half *w, __half *kv, int layer,
                                   int grid, int threads, hipStream_t s)
{
    const size_t lds = (size_t)P.lds_floats * 4;
    switch (P.dm.d) {
    case 64: hipLaunchKernelGGL(k_block_persistent<64>, dim3(grid), dim3(threads), lds, s, P, w, kv, layer); break;
    case 80: hipLaunchKernelGGL(k_block_persistent<80>, dim3(grid), dim3(threads), lds, s, P, w, kv, layer); break;
    case 128: hipLaunchKernelGGL(k_block_persistent<128>, dim3(grid), dim3(threads), lds, s, P, w, kv, layer); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// one thread block copies the by-value table into device memory
__global__ void k_store_layer_ptrs(LayerPtrs src, LayerPtrs *dst, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        dst->w[i] = src.w[i];
        dst->kv[i] = src.kv[i];
    }
}

hipError_t launch_store_layer_ptrs(const LayerPtrs &ptrs, LayerPtrs *dst, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_store_layer_ptrs, dim3(1), dim3(64), 0, s, ptrs, dst, n);
    return hipGetLastError();
}

hipError_t persistent_occupancy(int head_dim, int threads, size_t lds_bytes, int *blocks_per_cu)
{
    switch (head_dim) {
    case 64: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_block_persistent<64>, threads, lds_bytes);
    case 80: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_block_persistent<80>, threads, lds_bytes);
    case 128: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_block_persistent<128>, threads, lds_bytes);
    }
    return hipErrorInvalidValue;
}

// allow more than the default 64 KiB of dynamic LDS
hipError_t prepare_kernels(size_t lds_bytes)
{
    const int v = (int)lds_bytes;
    CFPP_TRY(hipFuncSetAttribute((const void *)k_phase_a, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_phase_c, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_phase_b<64>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_phase_b<80>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_phase_b<128>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_block_persistent<64>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_block_persistent<80>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    CFPP_TRY(hipFuncSetAttribute((const void *)k_block_persistent<128>, hipFuncAttributeMaxDynamicSharedMemorySize, v));
    return hipSuccess;
}

}  // namespace cfpp
