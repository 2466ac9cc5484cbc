// Projections of the prompt-sized path (paper Sec. 2.2 applied to hundreds of tokens): C[tokens][n] =
// A[tokens][K] . W[n][K]^T as LDS-tiled GEMMs on the matrix cores (v_mfma_f32_32x32x16_f16).
// Activations are two fp16 planes, head and remainder (half_split.h), each fed to the
// instruction in turn: the product of the fp32 values to rounding, fp32 accumulation.
//
//   k_pf_gemm<kPfIn>  : QKV rows and MLP-up rows of a layer, one launch (their output columns side by
//                       side); the epilogue completes the LayerNorm, rotates, appends, applies GELU
//   k_pf_gemm<kPfOut> : output projection and MLP-down as ONE product over the concatenated K
//                       ([attention | GELU(up)] . [W_dense | W_down]^T) + biases + residual
//   k_pf_reduce       : the parts of the first product, where its K is split over workgroups, added in
//                       order, then the same epilogue (the second one's: k_pf_row)
//
// Every sum has a fixed order: one bit pattern per build and pass size.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "prefill_device.h"
#include "lds_dma.h"

namespace cfpp {

typedef _Float16 pf_f16x8 __attribute__((ext_vector_type(8)));
typedef float pf_f32x16 __attribute__((ext_vector_type(16)));

enum { kPfIn = 0, kPfOut = 1 };
enum { kPfQkv = 0, kPfUp = 1 };                     // what follows the first product

// the LayerNorm, completed: inv (W (gamma x) - mu s) + c, with c = W beta + b from the packing
template <int EPI>
__device__ __forceinline__ float pf_complete(const PfParams &P, int row, int col, float val)
{
    const float2 rc = reinterpret_cast<const float2 *>(P.w + (EPI == kPfQkv ? P.lay.rc_qkv : P.lay.rc_up))[col];
    const float2 st = P.stats[row];
    return (val - st.x * rc.x) * st.y + rc.y;
}

// The element (row = token, col = output feature) with the completed value `val`;
// other: the completed value of the neighbouring column (col ^ 1) of the same row (QKV only:
// a rotation pair of the packed order sits in two adjacent columns, the first one even)
template <int EPI>
__device__ __forceinline__ void pf_store(const PfParams &P, int row, int col, float val, float other)
{
    const Dims &dm = P.dm;
    const int h = dm.h;
    if (EPI == kPfQkv) {
        const int pd = col / dm.d, i = col - pd * dm.d, nh = pd / 3, c = pd - 3 * nh;
        int dim = i;
        if (c < 2 && i < dm.r) {
            const float2 cs = P.rope[(size_t)(P.pos0 + row) * (dm.r >> 1) + (i >> 1)];
            if (i & 1) { val = val * cs.x + other * cs.y; dim = (i >> 1) + (dm.r >> 1); }
            else { val = val * cs.x - other * cs.y; dim = i >> 1; }
        }
        if (c == 0) P.q[(size_t)row * h + nh * dm.d + dim] = val;
        else P.kv[kv_offset(dm, c - 1, P.b, nh, dim, P.pos0 + row)] = __float2half_rn(val);
    } else {
        __half hi, lo;
        split_half(pf_gelu(val, dm.flags), hi, lo);
        const size_t at = pf_at(row, col, dm.f);
        P.m[at] = hi; P.m[at + kPfLo] = lo;
    }
}

// ---------------------------------------------------------------------------
// First row of a DMA instruction that takes `group` rows of an operand of `rows`: an instruction of a tile that overhangs
// the operand brings its last rows instead (what is made of them is never stored), so that no address leaves it.
// rows: a multiple of 128, group: at most 16
CFPP_HD int pf_dma_row(int row, int rows, int group) { return row < rows - group ? row : rows - group; }
template <int N>
__device__ __forceinline__ void pf_wait_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

template <int BM, int BN, int BK, int ST>
constexpr int pf_gemm_lds_bytes()
{
    return ST * (2 * BM + BN) * BK * 2;
}
constexpr int pf_per_cu(int lds) { return 160 * 1024 / lds > 3 ? 3 : 160 * 1024 / lds; }   // workgroups of a CU

// GEMM.  Workgroup: WM x WN wavefronts, tile BM tokens x BN output features, K in steps of BK through a ring of ST
// stages in LDS that is filled by DMA (memory -> LDS, no registers) up to ST - 1 steps ahead.  What bounds it, measured
// at 4096 tokens of the 2560-wide shape with parts switched off: matrix instructions alone 430 - 460 us of the second
// product's 541, the DMA alone 400 - 480; a CU's DMA rate is what is in flight (96 - 110 KB) over the latency of the
// slowest line of a step (about 2 us under load), not a bandwidth: 128-byte segments instead of 64, prefetching the
// weights' lines into the L2 (+ 5 % time) or K steps of 64 changed little.  Hence:
//   - tiles with few bytes per operation and a ring that fills the LDS (one or two workgroups to a CU), or three
//     workgroups of small tiles; which one: see pf_plan;
//   - a step's DMA instructions, its fragment reads and its matrix instructions are interleaved; the next K values'
//     fragments are read behind the first matrix instructions of the current ones, across the step's one barrier too;
//   - a wavefront owns BM / WM x BN / WN of the tile (32 x 160 ... 64 x 160): wide in the features, because an activation
//     fragment is two planes and a weight fragment one;
//   - rows of the activation buffers sit 256 bytes further apart than their values (a step reads one K offset of every
//     row: with strides of a multiple of 4 KiB those lines share memory channels: 594 -> 545 us, same product).
// Tiles are dealt so that consecutive numbers run on the same XCD (workgroup i runs on XCD i % 8), in groups of gm token
// tiles: an XCD works on a block of about gm x (its workgroups / gm) tiles and its L2 holds both operands' rows.
// splits > 1: workgroup z of a tile takes the z-th part of K and leaves its sums in part[z][row][col] (rows of whole
// token tiles); k_pf_reduce and k_pf_row add the parts in order and finish.
template <int FL, int BM, int BN, int BK, int ST, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN, pf_per_cu(pf_gemm_lds_bytes<BM, BN, BK, ST>()) * WM * WN / 4)
k_pf_gemm(PfParams P, int splits, int gm)
{
    constexpr int NT = 64 * WM * WN, NWV = WM * WN;
    constexpr int RB = BK * 2, PR = RB / 16, RU = 64 / PR;         // weights: bytes and 16-byte pieces of a row in LDS, rows of a DMA instruction
    constexpr int SUB = BK / 32, RBA = 128, RUA = 8;               // activations: 128-byte rows of 32 values (heads, remainders), SUB blocks of them
    constexpr int MT = BM / WM / 32, NTL = BN / WN / 32, KS = BK / 16;
    constexpr int NA1 = BM / RUA / NWV, NA = SUB * NA1, NW = (BN / RU + NWV - 1) / NWV, NLD = NA + NW;   // DMA instructions of a wavefront and step
    static_assert(BM % (RUA * NWV) == 0 && NWV % 2 == 0 && BN % RU == 0 && (BK == 32 || BN % (RU * NWV) == 0), "whole DMA instructions");
    constexpr int STAGE = 2 * BM * RB + BN * RB;
    constexpr int TS = 2 * kPfLo + 8, kScratch = NWV * 32 * TS * 2;   // epilogue: halves between rows of a wavefront's scratch, bytes of all
    static_assert(kScratch + BN * 8 <= ST * STAGE, "the epilogue's memory");
    extern __shared__ __align__(16) char pf_lds[];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char *)pf_lds;
    const Dims &dm = P.dm;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int h = dm.h, f = dm.f;
    const int ntn0 = FL == kPfIn ? (P.qkv ? (3 * h + BN - 1) / BN : 0) : (h + BN - 1) / BN;
    const int ntn = FL == kPfIn ? ntn0 + (P.up1 - P.up0 + BN - 1) / BN : ntn0;
    const int mt = (P.n_rows + BM - 1) / BM, tiles = ntn * mt, total = tiles * splits;
    const int per_xcd = (total + 7) >> 3;
    const int v = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (v >= total) return;                               // (whole workgroup)
    const int z = v / tiles, tile = v - z * tiles;
    // groups of gm token tiles by all feature tiles, token tiles fastest: what an XCD works on at a time is a block
    // of about gm x (its workgroups / gm) tiles
    const int grp = tile / (gm * ntn), in_grp = tile - grp * gm * ntn, gh = min(gm, mt - grp * gm);
    const int m0 = (grp * gm + in_grp % gh) * BM, tn = in_grp / gh;
    const bool up = FL == kPfIn && tn >= ntn0;
    const int n0 = up ? P.up0 + (tn - ntn0) * BN : tn * BN, N = FL == kPfIn ? (up ? P.up1 : 3 * h) : h;
    const int n_steps = (FL == kPfIn ? h : h + f) / BK, j_dense = h / BK;
    const int js = (int)((long long)n_steps * z / splits), je = (int)((long long)n_steps * (z + 1) / splits);

    const __half *a_0 = FL == kPfIn ? (up ? P.y2 : P.y1) : P.o;
    const __half *w_0 = P.w + (FL == kPfIn ? (up ? P.lay.w_up : P.lay.w_qkv) : P.lay.w_dense);
    const unsigned as0 = (unsigned)pf_row_halves(h) * 2u, as1 = (unsigned)pf_row_halves(f) * 2u;       // bytes between activation rows
    const unsigned abytes0 = (unsigned)P.rows * as0, wbytes0 = (unsigned)N * (unsigned)h * 2u;
    const unsigned abytes1 = (unsigned)P.rows * as1, wbytes1 = (unsigned)h * (unsigned)f * 2u;
    // A DMA instruction covers 8 rows x 128 bytes of the activations, or RU rows x RB bytes of the weights: lane l
    // brings a 16-byte piece of one row into place l, which is where the row's piece (place ^ swizzle(row)) belongs:
    // the fragment reads of 16 consecutive rows hit 64 different banks
    const int r16 = (RU * wave + lane / PR) & 15, sw = BK == 32 ? (r16 >> 2) & 3 : (r16 >> 1) & 7;
    const unsigned piece_w = (unsigned)(((lane % PR) ^ sw) * 16), piece_a = (unsigned)(((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) * 16);
    const unsigned vw0 = (unsigned)(lane / PR) * (unsigned)h * 2u + piece_w, vw1 = (unsigned)(lane / PR) * (unsigned)f * 2u + piece_w;
    const unsigned va0 = (unsigned)(lane >> 3) * as0 + piece_a, va1 = (unsigned)(lane >> 3) * as1 + piece_a;
    // instructions [i0, i1) of those that bring step j in, so that they can be spread between matrix instructions
    auto issue = [&](int j, int stage, int i0, int i1) {
        const bool second = FL == kPfOut && j >= j_dense;
        const unsigned jj = (unsigned)(second ? j - j_dense : j), width = (unsigned)(second ? f : h), as = second ? as1 : as0;
        const unsigned va = second ? va1 : va0, vw = second ? vw1 : vw0;
        const i32x4 ra = dma_rsrc(second ? P.m : a_0, second ? abytes1 : abytes0);
        const i32x4 rw = dma_rsrc(second ? P.w + P.lay.w_down : w_0, second ? wbytes1 : wbytes0);
        const unsigned dst = lds0 + (unsigned)stage * (unsigned)STAGE + 1024u * (unsigned)wave;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            if (i < i0 || i >= i1) continue;
            if (i < NA) {
                const int sub = i / NA1, u = (i % NA1) * NWV;
                lds_dma16(ra, dst + sub * BM * RBA + 1024u * u, va, (unsigned)pf_dma_row(m0 + RUA * (wave + u), P.rows, RUA) * as + (jj * SUB + sub) * 128u);
            } else {
                // (where the wavefronts do not divide the rows, the last ones bring the last rows a second time)
                const unsigned u = (i - NA + 1) * NWV <= BN / RU ? wave + (i - NA) * NWV : min(wave + (i - NA) * NWV, BN / RU - 1);
                const unsigned at = lds0 + (unsigned)stage * (unsigned)STAGE + 2 * BM * RB + 1024u * u, from = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)pf_dma_row(n0 + RU * (int)u, N, RU) * width * 2u + jj * RB));
                // with one token tile the weights are read once; the hint pays where an instruction takes whole lines (BK 64:
                // 37 tokens, hidden 4096: 130 -> 120 us per layer; on half lines, BK 32, it costs: 72 -> 77 at hidden 2560)
                if (BK == 64 && mt == 1) lds_dma16_once(rw, at, vw, from);
                else lds_dma16(rw, at, vw, from);
            }
        }
    };
    pf_f32x16 acc[MT][NTL];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NTL; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
    // fragment of this lane: row lane % 32 of an instruction tile, halves 8 * (lane / 32) .. + 7 of a step of 16
    const int fr = lane & 31, hf = lane >> 5, fsw = BK == 32 ? (fr >> 2) & 3 : (fr >> 1) & 7;
    const char *fa = pf_lds + wm * (BM / WM) * RBA, *fw = pf_lds + 2 * BM * RB + wn * (BN / WN) * RB;
    int oa[2], ol[2], ow[KS];                              // heads, remainders (of a block of 32 values), weights
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        oa[k] = fr * RBA + (((2 * k + hf) ^ ((fr >> 1) & 7)) * 16);
        ol[k] = fr * RBA + (((4 + 2 * k + hf) ^ ((fr >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ow[ks] = fr * RB + (((2 * ks + hf) ^ fsw) * 16);
    static_assert(KS % 2 == 0, "two fragment sets swap roles");
    struct Frag { pf_f16x8 ah[MT], al[MT], w[NTL]; } F[2];
    auto fetch = [&](Frag &g, int stage, int ks) {
        const char *pa = fa + stage * STAGE + (ks >> 1) * BM * RBA, *pw = fw + stage * STAGE;
#pragma unroll
        for (int t = 0; t < MT; ++t) g.ah[t] = *reinterpret_cast<const pf_f16x8 *>(pa + oa[ks & 1] + t * 32 * RBA);
#pragma unroll
        for (int t = 0; t < NTL; ++t) g.w[t] = *reinterpret_cast<const pf_f16x8 *>(pw + ow[ks] + t * 32 * RB);
#pragma unroll
        for (int t = 0; t < MT; ++t) g.al[t] = *reinterpret_cast<const pf_f16x8 *>(pa + ol[ks & 1] + t * 32 * RBA);
    };
#pragma unroll
    for (int s = 0; s < ST; ++s)
        if (js + s < je) issue(js + s, s, 0, NLD);
    if (js + ST - 1 < je) pf_wait_barrier<(ST - 1) * NLD>();
    else pf_wait_barrier<0>();
    fetch(F[0], 0, 0);
    int stage = 0, prev = ST - 1;                          // stage of step j; of step j - 1, free since the last barrier
    for (int j = js; j < je; ++j) {
        const int next = stage + 1 == ST ? 0 : stage + 1;
        const bool more = j > js && j - 1 + ST < je;       // (the prologue requested the first ST steps)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const Frag &g = F[ks & 1];
            constexpr int PER = (NLD + KS - 2) / (KS - 1);             // DMA instructions per instruction group (none in the last)
#pragma unroll
            for (int sl = 0; sl < 2 * MT; ++sl) {
                const int a = sl % MT;
#pragma unroll
                for (int b = 0; b < NTL; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(g.w[b], sl < MT ? g.ah[a] : g.al[a], acc[a][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (sl == 0) {
                    // the next group's fragments, behind this group's first instructions: the wait for this
                    // group's own (all that is outstanding at its start) then never includes them
                    if (ks + 1 < KS) {
                        fetch(F[(ks + 1) & 1], stage, ks + 1);
                    } else if (j + 1 < je) {
                        if (j + ST - 1 < je) pf_wait_barrier<(ST - 2) * NLD>();
                        else pf_wait_barrier<0>();
                        fetch(F[0], next, 0);
                    }
                }
                if (ks + 1 < KS) {
                    constexpr int SL = 2 * MT;
                    const int d0 = ks * PER + PER * sl / SL, d1 = ks * PER + PER * (sl + 1) / SL;
                    if (more && d0 < d1 && d0 < NLD) issue(j - 1 + ST, prev, d0, d1 < NLD ? d1 : NLD);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        prev = stage;
        stage = next;
    }
    // Weights are the instruction's first operand, so that this lane holds, per instruction tile, ONE token (lane % 32) and the
    // features 8 g + 4 (lane / 32) .. + 3, g < 4, side by side in its registers 4 g ..: a token's statistics are read once, four features
    // go out in one store, a rotation pair is the lane's own.  us per layer, a feature and 16 tokens to a lane (2-byte stores, a
    // statistics pair read per value) -> this: hidden 512, 4000 tokens 167 -> 143; 1536, 512 tokens 96.7 -> 89.9; 2560, 512 / 1024 /
    // 4000 tokens 199.6 -> 194.3 / 387 -> 375 / 1379 -> 1348; 4096, 2048 tokens 1539 -> 1495.  What follows the first product of 512
    // tokens at hidden 2560 is still some 15 of its 116 us (9.5 and 13 without the QKV and the MLP-up columns' part).
    const int t_lane = wm * (BM / WM) + (lane & 31), f_lane = 4 * (lane >> 5);      // token of the first instruction tile; first feature of g = 0
    if (splits > 1) {
        const int nall = FL == kPfIn ? 3 * h + f : h, c0 = up ? 3 * h : 0;
        // 32 tokens x 32 columns at a time through LDS that no other wavefront touches, so that whole 128-byte lines are stored:
        // 16 bytes of a token from each lane, four lines' quarters to a store, cost 0.5 .. 1 us a launch
        float *part = (FL == kPfIn ? P.part : P.part_out) + ((size_t)z * mt * BM + m0 + wm * (BM / WM)) * nall + c0;
        float *t = reinterpret_cast<float *>(pf_lds) + wave * 32 * (TS / 2);
        __syncthreads();                                   // the last step's fragments have been read: the memory is free
#pragma unroll
        for (int b = 0; b < NTL; ++b) {
            const int col = n0 + wn * (BN / WN) + b * 32;
            if (col >= N) break;                           // (uniform; N: a multiple of 128)
#pragma unroll
            for (int a = 0; a < MT; ++a) {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<f32x4 *>(t + (lane & 31) * (TS / 2) + 8 * g + f_lane) =
                        f32x4{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 8 * i + (lane >> 3), c = 4 * (lane & 7);
                    *reinterpret_cast<f32x4 *>(part + (size_t)(a * 32 + r) * nall + col + c) = *reinterpret_cast<const f32x4 *>(t + r * (TS / 2) + c);
                }
            }
        }
        return;
    }
    const float inv_d = __builtin_amdgcn_rcpf((float)dm.d);            // (column / d: the half keeps every quotient off a whole number)
    // What follows the product.  Nothing is exchanged between the wavefronts, so nobody waits for the slowest.
    float2 st[MT];                                         // mean and 1/sigma of the lane's tokens
    f32x4 *src = reinterpret_cast<f32x4 *>(pf_lds + kScratch);         // row constants of the tile's features, two features to a piece
    if (FL == kPfIn) {
#pragma unroll
        for (int a = 0; a < MT; ++a) st[a] = P.stats[min(m0 + t_lane + a * 32, P.n_rows - 1)];      // (rows past the pass's tokens are never stored)
        const f32x4 *rc = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float2 *>(P.w + (up ? P.lay.rc_up : P.lay.rc_qkv)) + n0);
        __syncthreads();                                   // the last step's fragments have been read: the memory is free
        for (int i = tid; i < BN / 2; i += NT) src[i] = rc[min(i, (N - n0) / 2 - 1)];
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < NTL; ++b) {
        const int cw = wn * (BN / WN) + b * 32, c0 = n0 + cw;
        if (c0 >= N) break;                                // (uniform; N: a multiple of 128)
        if (FL == kPfIn && up) {
            // MLP-up: 32 tokens x 32 columns at a time through 4.5 KB of LDS that no other wavefront touches, so that
            // whole 128-byte lines (32 heads, 32 remainders) are stored
            __half *t = reinterpret_cast<__half *>(pf_lds) + wave * 32 * TS;
#pragma unroll
            for (int a = 0; a < MT; ++a) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    union { __half h[4]; uint2 u; } hi, lo;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const f32x4 rc = src[(cw + 8 * g + f_lane) / 2 + j];
                        split_half(pf_gelu((acc[a][b][4 * g + 2 * j] - st[a].x * rc[0]) * st[a].y + rc[1], dm.flags), hi.h[2 * j], lo.h[2 * j]);
                        split_half(pf_gelu((acc[a][b][4 * g + 2 * j + 1] - st[a].x * rc[2]) * st[a].y + rc[3], dm.flags), hi.h[2 * j + 1], lo.h[2 * j + 1]);
                    }
                    __half *to = t + (lane & 31) * TS + 8 * g + f_lane;
                    *reinterpret_cast<uint2 *>(to) = hi.u;
                    *reinterpret_cast<uint2 *>(to + kPfLo) = lo.u;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int rl = i * 8 + (lane >> 3), row = m0 + wm * (BM / WM) + a * 32 + rl;
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(t + rl * TS + (lane & 7) * 8);
                    if (row < P.n_rows) *reinterpret_cast<u32x4 *>(P.m + pf_at(row, c0, f) + (lane & 7) * 8) = v;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (FL == kPfIn) {
            // QKV: four features are dimensions i .. i + 3 of one head's q, k or v (head sizes and i are multiples of 4); pairs
            // of the rotated part sit side by side
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = c0 + 8 * g + f_lane, pd = (int)(((float)col + 0.5f) * inv_d), i = col - pd * dm.d;
                const int nh = (int)(((float)pd + 0.5f) * (1.f / 3.f)), c = pd - 3 * nh, r = dm.r, half = r >> 1;
                const bool rot0 = c < 2 && i < r, rot1 = c < 2 && i + 2 < r;
                const f32x4 ra = src[(cw + 8 * g + f_lane) / 2], rb = src[(cw + 8 * g + f_lane) / 2 + 1];
                __half *kp = P.kv + kv_offset(dm, c > 0 ? c - 1 : 0, P.b, nh, 0, P.pos0);
                const unsigned slab = (unsigned)dm.max_seq * 16u;
#pragma unroll
                for (int a = 0; a < MT; ++a) {
                    const int row = m0 + t_lane + a * 32;
                    if (row >= P.n_rows) continue;
                    float v[4] = {(acc[a][b][4 * g] - st[a].x * ra[0]) * st[a].y + ra[1], (acc[a][b][4 * g + 1] - st[a].x * ra[2]) * st[a].y + ra[3],
                                  (acc[a][b][4 * g + 2] - st[a].x * rb[0]) * st[a].y + rb[1], (acc[a][b][4 * g + 3] - st[a].x * rb[2]) * st[a].y + rb[3]};
                    float *q = P.q + (unsigned)row * (unsigned)h + (unsigned)(nh * dm.d);
                    __half *kv = kp + (unsigned)row * 16u;
                    if (rot0) {                            // dimensions i / 2, i / 2 + half and, of the second pair, the next (or i + 2, i + 3)
                        const float2 *cs = P.rope + (unsigned)(P.pos0 + row) * (unsigned)half + (unsigned)(i >> 1);
                        const float2 s0 = cs[0];
                        const float x0 = v[0] * s0.x - v[1] * s0.y, x1 = v[1] * s0.x + v[0] * s0.y;
                        float x2 = v[2], x3 = v[3];
                        int d2 = i + 2, d3 = i + 3;
                        if (rot1) {
                            const float2 s1 = cs[1];
                            x2 = v[2] * s1.x - v[3] * s1.y; x3 = v[3] * s1.x + v[2] * s1.y;
                            d2 = (i >> 1) + 1; d3 = d2 + half;
                        }
                        const int d0 = i >> 1, d1 = d0 + half;
                        if (c == 0) {
                            q[d0] = x0; q[d1] = x1; q[d2] = x2; q[d3] = x3;
                        } else {
                            kv[(unsigned)(d0 >> 4) * slab + (d0 & 15)] = __float2half_rn(x0);
                            kv[(unsigned)(d1 >> 4) * slab + (d1 & 15)] = __float2half_rn(x1);
                            kv[(unsigned)(d2 >> 4) * slab + (d2 & 15)] = __float2half_rn(x2);
                            kv[(unsigned)(d3 >> 4) * slab + (d3 & 15)] = __float2half_rn(x3);
                        }
                    } else if (c == 0) {
                        *reinterpret_cast<f32x4 *>(q + i) = f32x4{v[0], v[1], v[2], v[3]};
                    } else {
                        uint2 o;
                        o.x = pf_pack2(v[0], v[1]); o.y = pf_pack2(v[2], v[3]);
                        *reinterpret_cast<uint2 *>(kv + (unsigned)(i >> 4) * slab + (i & 15)) = o;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            const bool last = P.layer == P.n_layers - 1;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = c0 + 8 * g + f_lane;
                const uint2 de = *reinterpret_cast<const uint2 *>(P.w + P.lay.b_dense + col), dn = *reinterpret_cast<const uint2 *>(P.w + P.lay.b_down + col);
                const float2 de0 = unpack_h2(de.x), de1 = unpack_h2(de.y), dn0 = unpack_h2(dn.x), dn1 = unpack_h2(dn.y);
                f32x4 x[MT];
#pragma unroll
                for (int a = 0; a < MT; ++a)
                    x[a] = *as_global(reinterpret_cast<const f32x4 *>(P.xres + (unsigned)min(m0 + t_lane + a * 32, P.n_rows - 1) * (unsigned)h + (unsigned)col));
#pragma unroll
                for (int a = 0; a < MT; ++a) {
                    const int row = m0 + t_lane + a * 32;
                    if (row >= P.n_rows) continue;
                    const unsigned at = (unsigned)row * (unsigned)h + (unsigned)col;
                    const f32x4 o{x[a][0] + ((acc[a][b][4 * g] + de0.x) + dn0.x), x[a][1] + ((acc[a][b][4 * g + 1] + de0.y) + dn0.y),
                                  x[a][2] + ((acc[a][b][4 * g + 2] + de1.x) + dn1.x), x[a][3] + ((acc[a][b][4 * g + 3] + de1.y) + dn1.y)};
                    if (last) {
                        uint2 p;
                        p.x = pf_pack2(o[0], o[1]); p.y = pf_pack2(o[2], o[3]);
                        *reinterpret_cast<uint2 *>(P.out + at) = p;
                    } else {
                        *reinterpret_cast<f32x4 *>(P.xnext + at) = o;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// the parts of the split first product (prows rows per part), added in order, then what follows it;
// a thread takes four consecutive columns of a row (two rotation pairs).  (The second product's parts
// are added by the kernel that prepares the next layer's input: k_pf_row.)
__global__ void __launch_bounds__(256) k_pf_reduce(PfParams P, int splits, int prows)
{
    const int nq = 3 * P.dm.h, N = nq + P.dm.f, n4 = N >> 2;
    const unsigned n_el = (unsigned)P.n_rows * (unsigned)n4;
    const size_t zstride = (size_t)prows * N;
    for (unsigned e = blockIdx.x * 256u + threadIdx.x; e < n_el; e += gridDim.x * 256u) {
        const int row = (int)(e / (unsigned)n4), col = (int)(e - (unsigned)row * (unsigned)n4) * 4;
        const float *p = P.part + (size_t)row * N + col;
        f32x4 s = *as_global(reinterpret_cast<const f32x4 *>(p));
        for (int z = 1; z < splits; ++z) s += *as_global(reinterpret_cast<const f32x4 *>(p + z * zstride));
        float v[4];
        if (col < nq) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = pf_complete<kPfQkv>(P, row, col + j, s[j]);
#pragma unroll
            for (int j = 0; j < 4; ++j) pf_store<kPfQkv>(P, row, col + j, v[j], v[j ^ 1]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) pf_store<kPfUp>(P, row, col - nq + j, pf_complete<kPfUp>(P, row, col - nq + j, s[j]), 0.f);
        }
    }
}

template <int FL, int BM, int BN, int BK, int ST, int WM, int WN>
static hipError_t pf_launch(const PfParams &P, const PfPlan &pl, hipStream_t s)
{
    const int h = P.dm.h, f = P.dm.f, splits = pl.splits;
    const int ntn = FL == kPfIn ? (P.qkv ? (3 * h + BN - 1) / BN : 0) + (P.up1 - P.up0 + BN - 1) / BN : (h + BN - 1) / BN;
    const int mt = (P.n_rows + BM - 1) / BM, nall = FL == kPfIn ? 3 * h + f : h;
    // the parts of a split product, [splits][mt * BM][all columns] floats, must fit what the scratch holds for them
    if (splits > 1 && (size_t)splits * mt * BM * nall * sizeof(float) > (FL == kPfIn ? P.part_bytes : P.part_out_bytes))
        return hipErrorInvalidValue;
    constexpr int lds = pf_gemm_lds_bytes<BM, BN, BK, ST>();
    const hipError_t e = hipFuncSetAttribute((const void *)k_pf_gemm<FL, BM, BN, BK, ST, WM, WN>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_pf_gemm<FL, BM, BN, BK, ST, WM, WN>), dim3((ntn * mt * splits + 7) / 8 * 8), dim3(64 * WM * WN), lds, s, P,
                       splits, BM == 256 ? 4 : 8);
    if (FL == kPfIn && splits > 1) {
        const size_t n_el = (size_t)P.n_rows * (nall / 4);
        hipLaunchKernelGGL(k_pf_reduce, dim3((unsigned)((n_el + 255) / 256)), dim3(256), 0, s, P, splits, mt * BM);
    }
    return hipSuccess;
}

// Tile and splits of K of a product.  No tile is best everywhere: what a CU does is whole tiles, so that the
// best one is the one whose tiles (times splits) fill the 256 CUs evenly, and a big tile moves fewer bytes per
// operation but finishes in one long epilogue.  The choice is the least estimate of
//     most tiles of a CU x (K / 32 / splits x step + epilogue)  [where several tiles share a CU: at least
//     rounds x K / 32 / splits x lone_step]
//     + (split: the parts written and read again)
// The constants are a least-squares fit in us to 1500 timings of one product alone (hidden 512 .. 4096, 8 .. 4096 tokens,
// every tile, splits 1 .. 16): they order the choices, and pick within 0.8 % of the fastest measured combination in the mean,
// 7.5 % at worst; inside a layer a product takes longer than its estimate (512 tokens: 106 us, estimate 76).
// Measured per layer (attention and LayerNorm included), before this kernel -> now: hidden 2560: 100 tokens 144 -> 103,
// 512: 303 -> 224, 4096: 2345 -> 1528; hidden 4096, 1531 tokens: 1810 -> 1203.  (Up to 64 tokens: pf_plan_short.)
constexpr int kPfCus = 256;
struct PfTileCost { int bm, bn, bk, per_cu; float step, lone_step, epi_in, epi_out; };
constexpr int kPfTile32x128 = 7, kPfTile64x256 = 8;    // (up to 64 tokens: pf_plan_short)
constexpr int kPfTile128x160 = 9, kPfTile128x128 = 10, kPfTile128x192 = 11, kPfTile128x256 = 12, kPfTile128x96 = 13;   // (65 .. 1024 tokens: pf_plan_middle)
static const PfTileCost kPfTiles[kPfTileKinds] = {
    {64, 128, 64, 1, 0.26f, 0.f, 3.74f, 2.19f},
    {64, 128, 32, 3, 0.25f, 0.37f, 0.01f, 1.13f},
    {128, 128, 32, 2, 0.36f, 0.46f, 3.17f, 2.15f},
    {128, 320, 32, 1, 0.88f, 0.f, 5.51f, 3.99f},
    {256, 192, 32, 1, 0.92f, 0.f, 9.92f, 4.42f},
    {256, 256, 32, 1, 1.10f, 0.f, 14.67f, 5.02f},
    {256, 320, 32, 1, 1.34f, 0.f, 27.44f, 6.68f},
    {32, 128, 64}, {64, 256, 64},
    {128, 160, 32, 2}, {128, 128, 64, 1}, {128, 192, 32, 1}, {128, 256, 32, 1}, {128, 96, 64, 1},
};

// Up to 64 tokens a product is its weights' way from memory, once.  One token tile of 32 or 64 rows (the activations
// of a tile are as many bytes as twice its rows of weights); K steps of 64, whole lines; and the 256 CUs filled once, by
// the wider tile of 64 tokens or by splitting K: the first product at most three ways (its parts cost a launch that adds them),
// the second up to sixteen (they are added where the next layer's input is made).  us per layer, least estimate above -> this:
// hidden 2560: 37 tokens 73.3 -> 66.0, 64 tokens 76.0 -> 71; hidden 4096, 20 tokens 129 -> 107.  (Most such passes run the narrow
// products now: pf_plan_narrow.  A tile of 32 x 256 left with them: no pass on 256 CUs took it any more.)
// False where that leaves half the CUs without a tile of 64 (hidden 512, 40 tokens: 31 us, 27 by the estimate).
static bool pf_plan_short(const PfParams &P, bool in, size_t part_bytes, PfPlan *plan)
{
    const int h = P.dm.h, f = P.dm.f, nall = in ? 3 * h + f : h;
    const bool low = P.n_rows <= 32;
    const int kinds[2] = {low ? kPfTile32x128 : 0, kPfTile64x256};
    PfPlan best = {kinds[0], 1};
    int most = 0;
    for (int i = 0; i < (in && !low ? 2 : 1); ++i) {
        const PfTileCost &t = kPfTiles[kinds[i]];
        const int tiles = in ? (3 * h + t.bn - 1) / t.bn + (f + t.bn - 1) / t.bn : (h + t.bn - 1) / t.bn;
        for (int sp = 1; sp <= (in ? 3 : 16); ++sp) {
            if (sp > 1 && (tiles * sp > kPfCus || (size_t)sp * t.bm * nall * sizeof(float) > part_bytes)) break;
            const int wgs = tiles < kPfCus ? tiles * sp : kPfCus;
            if (wgs > most || (wgs == most && sp < best.splits)) { most = wgs; best.tile = kinds[i]; best.splits = sp; }
        }
    }
    *plan = best;
    return low || most >= kPfCus / 2;
}

static PfPlan pf_plan(const PfParams &P, bool in, size_t part_bytes, float *cost_out)
{
    PfPlan few;
    if (P.n_rows <= 64 && pf_plan_short(P, in, part_bytes, &few)) {
        *cost_out = 0.f;
        return few;
    }
    const int h = P.dm.h, f = P.dm.f, nall = in ? 3 * h + f : h;
    const float steps = (float)(in ? h : h + f) / 32.f;
    PfPlan best = {0, 1};
    float best_cost = 1e30f;
    for (int k = 0; k < kPfTile32x128; ++k) {
        const PfTileCost &t = kPfTiles[k];
        if (in && t.bn == 320 && t.bm == 256) continue;    // (left to pf_plan_long)
        const int mt = (P.n_rows + t.bm - 1) / t.bm;
        const int ntn = in ? (3 * h + t.bn - 1) / t.bn + (f + t.bn - 1) / t.bn : (h + t.bn - 1) / t.bn;
        for (int sp = 1; sp <= 16; ++sp) {
            if (sp > 1 && ((long long)mt * ntn * sp > 8 * kPfCus || (size_t)sp * mt * t.bm * nall * sizeof(float) > part_bytes)) break;
            const int wgs = mt * ntn * sp, per = (wgs + kPfCus - 1) / kPfCus, rounds = (wgs + kPfCus * t.per_cu - 1) / (kPfCus * t.per_cu);
            const float busy = per * (steps / sp) * t.step, lone = rounds * (steps / sp) * t.lone_step;
            float cost = (busy > lone ? busy : lone) + per * (in && sp == 1 ? t.epi_in : t.epi_out);
            if (sp > 1) cost += 0.89f + 1.12e-6f * sp * P.n_rows * (float)nall;
            if (cost < best_cost) { best_cost = cost; best.tile = k; best.splits = sp; }
        }
    }
    *cost_out = best_cost;
    return best;
}

static void pf_plan_ends(PfParams &P)
{
    P.up_cut = P.dm.f;
    P.row_fused = P.plan_out.splits > 1 && P.part_out == P.q;
    const int bm = kPfTiles[P.plan_out.tile].bm;
    P.part_out_stride = (size_t)((P.n_rows + bm - 1) / bm * bm) * P.dm.h;
}

void pf_plan_pass(PfParams &P)
{
    float cost, cost_y;
    P.plan_in = pf_plan(P, true, P.part_bytes, &cost);
    // The second product's parts lie behind y2, where the kernel that adds them can leave the next layer's y1 and
    // y2; or, where that space is too small for the splits that pay, from y1 on, with the LayerNorm in a launch of
    // its own again (10 us at 512 tokens and below, 24 at 4096).  An unsplit product has that launch as well.
    const size_t ahead = (size_t)((char *)P.q - (char *)P.y1);
    const float ln = 8.f + 1.6e-6f * P.n_rows * (float)P.dm.h;
    P.part_out = reinterpret_cast<float *>(P.q);
    P.plan_out = pf_plan(P, false, P.part_out_bytes, &cost);
    if (P.plan_out.splits == 1) cost += ln;
    const PfPlan wide = pf_plan(P, false, P.part_out_bytes + ahead, &cost_y);
    if (cost_y + ln < cost) {
        P.plan_out = wide;
        P.part_out = reinterpret_cast<float *>(P.y1);
        P.part_out_bytes += ahead;
    }
    pf_plan_ends(P);
}

// Passes of 65 .. 1024 tokens: five more tiles of 128 tokens, where they beat the plan above.  With one or two token tiles
// a product of few tokens is few workgroups with a whole K each, and what counts is that they come to nearly the number of
// CUs: 96, 160 (two workgroups to a CU), 192 or 256 features (a deeper ring); and K steps of 64 values - whole lines of weights, half
// the barriers (loads of 64-byte segments run at half the rate of 128: 69 and 133 KB/us a CU) - where a CU has one workgroup.  Chosen by an estimate of the same form whose constants, in us, are
// fitted to timings of whole layers (hidden 512 .. 4096, 70 .. 1024 tokens, 5500 of them, 2.4 % of a layer rms); taken where it is 2 us and
// 2 % below that of the plan above.  us per layer, before -> now: hidden 2560: 256 tokens 148 -> 130, 512 207 -> 200; hidden 4096: 96
// 179 -> 154; hidden 1536, 512 99 -> 95.  The timings were of three layers, whose weights stay in the Infinity Cache below hidden 1800 or
// so, and there the estimate prices a split of the first product too low: with 900 MB of layers a whole one that is cut in two
// loses 4.5 .. 12 % of a layer at every size of 15 (1792, 128 tokens 54.5 -> 60.6; 2304, 100 tokens 71.2 -> 76.5).  So K is
// split only where the plan above splits it; of the 188 other changes timed that way none is slower (0 .. 19 % of a layer faster).
struct PfLayerCost { float step, lone_step, epi_in, epi_out; };
static const PfLayerCost kPfLayerCosts[kPfTileKinds] = {
    {0.271f, 0.000f, 4.96f, 1.94f},
    {0.237f, 0.336f, 0.98f, 0.89f},
    {0.325f, 0.435f, 6.76f, 2.00f},
    {0.809f, 0.000f, 9.63f, 4.32f},
    {0.849f, 0.000f, 13.36f, 5.07f},
    {1.007f, 0.000f, 17.27f, 6.35f},
    {1.236f, 0.000f, 25.35f, 7.53f},
    {}, {},
    {0.405f, 0.551f, 8.04f, 2.47f},
    {0.376f, 0.000f, 10.05f, 3.39f},
    {0.566f, 0.000f, 5.09f, 3.08f},
    {0.693f, 0.000f, 6.71f, 3.74f}, {},
};
static float pf_layer_cost(const PfParams &P, bool in, int kind, int sp)
{
    const PfTileCost &t = kPfTiles[kind];
    const PfLayerCost &c = kPfLayerCosts[kind];
    const int h = P.dm.h, f = P.dm.f, mt = (P.n_rows + t.bm - 1) / t.bm;
    const int ntn = in ? (3 * h + t.bn - 1) / t.bn + (f + t.bn - 1) / t.bn : (h + t.bn - 1) / t.bn;
    const int wgs = mt * ntn * sp, per = (wgs + kPfCus - 1) / kPfCus, rounds = (wgs + kPfCus * t.per_cu - 1) / (kPfCus * t.per_cu);
    const float steps = (float)(in ? h : h + f) / 32.f / sp, nall = (float)(in ? 3 * h + f : h);
    const float busy = per * steps * c.step, lone = rounds * steps * c.lone_step;
    float cost = busy > lone ? busy : lone;
    if (!in) cost += per * c.epi_out;
    else if (sp == 1) cost += per * c.epi_in;
    if (sp > 1) cost += in ? 4.32f + 8.33e-07f * sp * P.n_rows * nall : 0.08f + 9.54e-07f * sp * P.n_rows * nall;
    return cost;
}
void pf_plan_middle(PfParams &P)
{
    if (P.n_rows <= 64 || P.n_rows > 1024) return;
    for (int in = 1; in >= 0; --in) {
        PfPlan &plan = in ? P.plan_in : P.plan_out;
        const size_t room = in ? P.part_bytes : P.part_out_bytes;
        const bool whole = plan.splits == 1;
        const float was = pf_layer_cost(P, in, plan.tile, plan.splits);
        float best = 0.98f * was - 2.f;
        for (int k = kPfTile128x160; k <= kPfTile128x256; ++k) {
            if (!in && (k == kPfTile128x160 || k == kPfTile128x256)) continue;     // (never the least there: not built)
            const int mt = (P.n_rows + 127) / 128, nall = in ? 3 * P.dm.h + P.dm.f : P.dm.h;
            for (int sp = 1; sp <= (in ? 4 : 16); ++sp) {
                if (sp > 1 && ((in && (k != kPfTile128x128 || whole)) || (size_t)sp * mt * 128 * nall * sizeof(float) > room)) break;
                if ((in ? P.dm.h : P.dm.h + P.dm.f) / kPfTiles[k].bk < sp) break;
                const float cost = pf_layer_cost(P, in, k, sp);
                if (cost < best) { best = cost; plan.tile = k; plan.splits = sp; }
            }
        }
    }
    // The first product with tiles of 128 x 96, K in steps of 64 and whole, one to a CU, where tiles of 64 x 128 no longer are: from
    // there on the plan above pairs these, or splits K into more workgroups than CUs, and its estimate (of products whose weights
    // are in the Infinity Cache in part) does not see what that costs.  us per layer, 900 MB of layers so that weights come from
    // memory, plan above -> this, by workgroups of 64 x 128 tiles: 252 .. 255: hidden 1536, 192 tokens 55.0 -> 60.6, 2304, 96 tokens
    // 73.4 -> 75.1, 2176 / 4352 (hidden / ffn), 176 tokens 64.7 -> 71.2; 260 .. 280: 1664 / 3328, 224 tokens 61.9 -> 60.6, 2432, 96
    // tokens 94.3 -> 79.1, 1664, 176 tokens 68.5 -> 65.9, 1280, 256 tokens 56.7 -> 55.9, 2560, 96 tokens 104.2 -> 86.6; above: 1536, 224
    // tokens 70.9 -> 65.0, 4096 / 8192, 96 tokens 139 -> 117.  Of 90 timed sizes above the line (hidden 1280 .. 4096) none was slower, of
    // 108 below it 93 were.  Shorter products lose more of a pair's gain to their ends: below hidden 1280 the line lies higher (264:
    // 1024 / 8192, 190 tokens 50.8 -> 52.0, 768 / 6144, 200 tokens 44.3 -> 45.2; 308 and 352: 896 / 7168 and 1024 / 8192, 200 tokens 52.0 -> 49.2,
    // 57.4 -> 53.8), and with more than 256 tokens either may be ahead (512, 640 tokens 43.5 -> 45.3, 1024, 384 tokens 55.0 -> 53.8).
    const int h = P.dm.h, f = P.dm.f, wgs64 = (P.n_rows + 63) / 64 * ((3 * h + f) / 128);
    const int wgs96 = (P.n_rows + 127) / 128 * ((3 * h + 95) / 96 + (f + 95) / 96);
    if (P.n_rows <= 256 && wgs64 > (h >= 1280 ? kPfCus : kPfCus + 32) && wgs96 <= kPfCus) P.plan_in = PfPlan{kPfTile128x96, 1};
    pf_plan_ends(P);
}

// The first product of a long pass: what a CU does is whole tiles, and 2.1 or 4.4 rounds of large ones take as long as 3 or 5.  So it may
// run as two launches: a whole number of rounds of large tiles (QKV and most of MLP-up), and the rest of MLP-up in smaller ones
// that fill one round more; and 256 x 320 tiles are among the large ones (with a feature and 16 tokens to a lane their epilogues spilled
// registers; now they don't).  Chosen by an estimate of
//     rounds x (K / 32 x step + epilogue) + kPfCutLaunch for a second launch
// whose constants, in us, are fitted to timings of whole layers with every one of these tiles (hidden 1280 .. 4096, 600 .. 4096 tokens, 352 of
// them, 1.1 % rms; the tile it picks is 0.1 % from the fastest in the mean, 1.9 % at worst).  It prices the last, partly filled round of a launch
// too high (fewer CUs, more power and bandwidth to each) and the gap between two launches too low: 12 us for the second one, and 2.5 %
// and 2 us, put the line where 130 random sizes had it (with 4 us 1536, 3198 tokens 481 -> 494).  us per layer, plan above -> this: whole: hidden
// 2560, 1000 tokens 377 -> 357, 3120 1153 -> 1121; 1536, 3482 541 -> 516; 3072, 1690 824 -> 774; 4096, 3362 2731 -> 2613; in two: 2560, 2880 tokens
// 1020 -> 983, 4096 1383 -> 1361; 2048, 3573 888 -> 832; 4096, 1531 behind 700 1192 -> 1185, 1670 1380 -> 1313.  Of the 130 sizes none lost more
// than the runs of one side differ (1 %).  128 x 128 tiles are never the second launch: the estimate would name them at one size in eighty, and of 32 such
// (hidden 2304 .. 4096, 1410 .. 4032 tokens) they were 0.0 % from the others in the mean, -1.1 to 0.9 % in single ones.
struct PfLongCost { float step, epi; };
constexpr float kPfCutLaunch = 12.f;
static const PfLongCost kPfLongCosts[kPfTileKinds] = {
    {}, {}, {}, {0.786f, 8.5f}, {0.891f, 7.6f}, {1.089f, 10.5f}, {1.291f, 14.9f}, {}, {}, {0.399f, 3.3f}, {0.375f, 6.9f}, {0.530f, 5.5f}, {0.652f, 6.1f}, {},
};
void pf_plan_long(PfParams &P)
{
    if (P.plan_in.splits != 1 || P.n_rows <= 512 || kPfLongCosts[P.plan_in.tile].step == 0.f) return;
    const int h = P.dm.h, f = P.dm.f;
    auto columns = [](int n, int bn) { return (n + bn - 1) / bn; };
    // `wide`: columns of tiles
    auto cost = [&](int kind, int wide) {
        const PfTileCost &t = kPfTiles[kind];
        const int wgs = (P.n_rows + t.bm - 1) / t.bm * wide, rest = wgs % (kPfCus * t.per_cu);
        float rounds = (float)(wgs / (kPfCus * t.per_cu) * t.per_cu);
        if (rest > 0) rounds += t.per_cu == 1 ? 1.f : rest <= kPfCus ? 1.36f : 2.f;        // (128 x 160, two to a CU: one alone is faster, by 1.36)
        return rounds * ((float)h / 32.f * kPfLongCosts[kind].step + kPfLongCosts[kind].epi);
    };
    const int bn0 = kPfTiles[P.plan_in.tile].bn;
    float best = cost(P.plan_in.tile, columns(3 * h, bn0) + columns(f, bn0)) * 0.975f - 2.f;
    for (int k = 0; k < kPfTileKinds; ++k) {
        if (kPfLongCosts[k].step == 0.f) continue;
        const PfTileCost &t = kPfTiles[k];
        const int mt = (P.n_rows + t.bm - 1) / t.bm, nq = columns(3 * h, t.bn);
        const float whole = cost(k, nq + columns(f, t.bn));
        if (whole < best) { best = whole; P.plan_in.tile = k; P.up_cut = f; }
        if (t.per_cu > 1) continue;
        for (int r = 1; r * kPfCus < mt * (nq + columns(f, t.bn)); ++r) {
            const int cut = (r * kPfCus / mt - nq) * t.bn / kPfTile * kPfTile;
            if (cut <= 0 || cut >= f) continue;
            const float first = cost(k, nq + columns(cut, t.bn)) + kPfCutLaunch;
            for (int j = 0; j < kPfTileKinds; ++j) {
                if (kPfLongCosts[j].step == 0.f || j == kPfTile128x128) continue;
                const float both = first + cost(j, columns(f - cut, kPfTiles[j].bn));
                if (both < best) { best = both; P.plan_in.tile = k; P.up_cut = cut; P.up_tile = j; }
            }
        }
    }
}

#ifdef CFPP_PROFILE
__global__ void __launch_bounds__(256) k_debug_gelu(const float *z, float *epilogue, float *library, int n, int flags)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    epilogue[i] = pf_gelu(z[i], flags);
    library[i] = gelu_act(z[i], flags);
}
hipError_t launch_debug_gelu(const float *z, float *epilogue, float *library, int n, int flags, hipStream_t s)
{
    hipLaunchKernelGGL(k_debug_gelu, dim3((n + 255) / 256), dim3(256), 0, s, z, epilogue, library, n, flags);
    return hipGetLastError();
}

void pf_describe_long(const PfParams &P, int plan[5], int past[2])
{
    const int h = P.dm.h, f = P.dm.f;
    const PfTileCost &a = kPfTiles[P.plan_in.tile], &b = kPfTiles[P.up_tile];
    auto reach = [](int from, int to, const PfTileCost &t) {           // of a matrix's rows [from, to)
        const int ru = 1024 / (2 * t.bk);
        int w = 0;
        for (int u = from; u < from + (to - from + t.bn - 1) / t.bn * t.bn; u += ru) w = max(w, pf_dma_row(u, to, ru) + ru - to);
        return w;
    };
    plan[0] = a.bm; plan[1] = a.bn; plan[2] = P.up_cut;
    plan[3] = P.up_cut < f ? b.bm : 0; plan[4] = P.up_cut < f ? b.bn : 0;
    past[0] = max(reach(0, 3 * h, a), reach(0, P.up_cut, a));
    past[1] = P.up_cut < f ? reach(P.up_cut, f, b) : 0;
}

void pf_describe_plan(const PfParams &P, int plan[8], int past[4])
{
    for (int k = 0; k < 2; ++k) {
        const PfPlan &pl = k ? P.plan_out : P.plan_in;
        const int bm = kPfTiles[pl.tile].bm, bn = kPfTiles[pl.tile].bn, ru = 1024 / (2 * kPfTiles[pl.tile].bk), h = P.dm.h, f = P.dm.f;
        plan[4 * k] = bm; plan[4 * k + 1] = bn; plan[4 * k + 2] = kPfTiles[pl.tile].bk; plan[4 * k + 3] = pl.splits;
        // rows past the operand that the last instruction of a tile reaches, as k_pf_gemm's issue() forms them: the
        // first product's matrices have 3 h and f rows, the second's h
        int a = 0, w = 0;
        for (int u = 0; u < (P.n_rows + bm - 1) / bm * bm; u += 8) a = max(a, pf_dma_row(u, P.rows, 8) + 8 - P.rows);
        const int n[2] = {k ? h : 3 * h, k ? h : f};
        for (int i = 0; i < 2; ++i)
            for (int u = 0; u < (n[i] + bn - 1) / bn * bn; u += ru) w = max(w, pf_dma_row(u, n[i], ru) + ru - n[i]);
        past[2 * k] = a; past[2 * k + 1] = w;
    }
}
#endif

template <int FL>
static hipError_t pf_gemm(const PfParams &P, const PfPlan &pl, hipStream_t s)
{
    switch (pl.tile) {
    case 0: return pf_launch<FL, 64, 128, 64, 4, 2, 2>(P, pl, s);
    case 1: return pf_launch<FL, 64, 128, 32, 3, 2, 2>(P, pl, s);
    case 2: return pf_launch<FL, 128, 128, 32, 3, 2, 2>(P, pl, s);
    case 3: return pf_launch<FL, 128, 320, 32, 4, 4, 2>(P, pl, s);
    case 4: return pf_launch<FL, 256, 192, 32, 3, 4, 2>(P, pl, s);
    case 5: return pf_launch<FL, 256, 256, 32, 3, 4, 2>(P, pl, s);
    case 6: return pf_launch<FL, 256, 320, 32, 3, 4, 2>(P, pl, s);
    case kPfTile32x128: return pf_launch<FL, 32, 128, 64, 3, 1, 4>(P, pl, s);
    case kPfTile64x256: if (FL == kPfIn) return pf_launch<kPfIn, 64, 256, 64, 3, 1, 4>(P, pl, s); break;
    case kPfTile128x160: if (FL == kPfIn) return pf_launch<kPfIn, 128, 160, 32, 3, 4, 1>(P, pl, s); break;
    case kPfTile128x128: return pf_launch<FL, 128, 128, 64, 3, 2, 2>(P, pl, s);
    case kPfTile128x96: if (FL == kPfIn) return pf_launch<kPfIn, 128, 96, 64, 3, 4, 1>(P, pl, s); break;
    case kPfTile128x192: return pf_launch<FL, 128, 192, 32, 5, 4, 2>(P, pl, s);
    case kPfTile128x256: if (FL == kPfIn) return pf_launch<kPfIn, 128, 256, 32, 4, 4, 2>(P, pl, s); break;
    }
    return hipErrorInvalidValue;
}

hipError_t launch_pf_gemm_in(const PfParams &P, hipStream_t s)
{
    PfParams Q = P;
    Q.qkv = true; Q.up0 = 0; Q.up1 = P.up_cut;
    const hipError_t e = pf_gemm<kPfIn>(Q, P.plan_in, s);
    if (e != hipSuccess || P.up_cut == P.dm.f) return e;
    Q.qkv = false; Q.up0 = P.up_cut; Q.up1 = P.dm.f;
    return pf_gemm<kPfIn>(Q, PfPlan{P.up_tile, 1}, s);
}
hipError_t launch_pf_gemm_out(const PfParams &P, hipStream_t s) { return pf_gemm<kPfOut>(P, P.plan_out, s); }

}  // namespace cfpp
