// Attention of the batched path (narrow_gemm.hip, lone_gemm.hip), and MLP-down in the same launch.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "attention_common.h"
#include "mlp_down.h"

namespace cfpp {

// The attention of several sequences in one launch.  P holds the parameters of the first
// sequence; sequence i follows at the workspace's usual strides.  A workgroup (4 wavefronts,
// several to a CU) takes one piece of ONE head of one sequence: every head of sequence i is cut
// into 1 + spare * rows_i / rows_all pieces, worked out by every workgroup from the positions in
// device memory (the grid is the most that can come out; what is over leaves at once); of a prompt group, into `spare`.  So a
// short sequence is as many workgroups as it has heads, and none does several heads one after
// the other: dealing 256 workgroups of 512 threads to the sequences by length left the heads of
// a short one to one or two of them, a staging, merge and hand-over (about 1.2 us) per head.
// Wavefronts interleave the piece's rows (PPW positions each), two rows in flight; the running
// softmax is per lane group and merged lane -> wavefront -> workgroup -> head, each in a fixed
// order; the workgroup that delivers a head's last piece adds the pieces in order.  The new token's
// K and V row is read from the cache like the others (the launch before this one wrote it).
// STREAM: non-temporal loads (every row is read once); without: a group of prompt tokens, whose
// queries read the same rows (attn_bstep = 0).
// Workgroups dealt beyond one per head and sequence, and the fewest rows worth a piece.  us per step and layer, before
// -> with pieces of 8 / 16 / 32 rows: five sequences of 37 .. 2048 positions (hidden 2560) 85.0 -> 65.9 / 65.7 / 63.6;
// 8 prompt tokens behind 1000: 67.3 -> 70.5 / 66.4 / 64.2; two sequences of 8000: 80.0 -> 81.8 / 79.4 / 78.9. 
// Spare ones of sequences with K/V rows of their own: 640, shared out by rows and rounded down per sequence, so that with one
// per head it comes to 650 .. 900 workgroups of about one size for up to 32 heads, about what is resident at 3 a CU.  Chosen at 32 heads and 8
// sequences: one block of hidden 4096, 3219 .. 7696 positions, 256 / 512 / 640 / 1024 / 2048 spare ones: 224.4 / 219.4 /
// 218.2 / 222.7 / 223.7 us (218.2 with the 256 workgroups of before); of 1024 .. 8192 positions 640 / 1024 / 2048: 231.8 /
// 232.0 / 230.4 (234 .. 236 before).  Elsewhere 640 was held against the kernels of before only, us per whole step: 8 heads, 4 layers,
// 2 sequences of 6000 .. 8000 183 -> 157, 8 of 2000 190 -> 169; 24 heads, 4 layers 245 -> 232, 266 -> 257; 32 heads of 80,
// 2 layers 168 -> 156, 182 -> 178.
// A prompt group's queries share their rows and don't stream: every head of a query is cut into as many pieces as come to 256 workgroups, one at
// least, and the host, which knows the group's positions, makes the grid no larger.  Before, 1024 spare ones and a grid for the longest context, in which
// hundreds of workgroups left at once ahead of MLP-down's.  us a layer, before -> this, room for 4100 positions: 8 tokens of hidden 1536
// behind 20 / 400 24.0 / 25.0 -> 21.1 / 22.5, 2560 39.2 / 39.5 -> 36.3 / 38.1, 4096 behind 880 86.5 -> 77.3; 8 heads of 128, behind 2500
// 27.1 -> 24.7; 512 or 1024 workgroups of pieces: 0 .. 10 % more where a head has two or more.
// A head's pieces leave the last kDownParts of its part_slots to MLP-down.
constexpr int kAttnSpareGroups = 640, kAttnSharedGroups = 256, kAttnPieceRows = 32;
// Up to four sequences, or tokens of a group, leave workgroups to spare: up to eight pieces of half as many rows.  us a block, 32 rows -> 16:
// hidden 2560, one sequence of 1000 / 2000 / 4000 41.3 -> 39.5 / 43.4 -> 41.0 / 45.4 -> 43.7, three of 500 .. 1000 42.9 -> 41.8;
// hidden 4096, four of 20 .. 2000 85.7 -> 83.6; but five of 37 .. 2048 45.6 -> 47.4, prompt groups of 8 47.0 -> 47.9, and 16 pieces
// of one sequence of 8000 49.7 -> 50.4.  Groups of 2 tokens, which are as few: hidden 2560 behind 880 39.2 -> 36.9, 3072 51.4 -> 50.0.
constexpr int kAttnFew = 4;
CFPP_HD int attn_pieces(int rows, bool few)
{
    const int n = (rows + kAttnPieceRows - 1) / kAttnPieceRows, half = (rows + kAttnPieceRows / 2 - 1) / (kAttnPieceRows / 2);
    return !few || n >= 8 ? n : half < 8 ? half : 8;
}

template <int D, bool STREAM, bool ONE>
__global__ void __launch_bounds__(kAttnBatchThreads, 3)
k_attention_batched(StepParams P, int nb, int spare, bool few, const __half *kv, DownPlan down)
{
    extern __shared__ __align__(16) char at_lds[];
    if ((int)blockIdx.x >= down.first) {
        mlp_down<ONE>(P, down, (int)blockIdx.x - down.first, nb, at_lds);
        return;
    }
    using A = AttnShape<D>;
    constexpr int LPP = A::LPP, PPW = A::PPW, NP = A::NP, NV = A::NV, NE = (D + 63) / 64, NW = kAttnBatchThreads / 64;
    float *qs = reinterpret_cast<float *>(at_lds), *wp = qs + D, *wm = wp + NW * D, *wl = wm + NW;
    static_assert((D + NW * D + 2 * NW) * 4 <= down_lds<ONE>(), "");
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
            const int n = min(min(STREAM ? 1 + (int)((float)rows[i] * share) : spare, attn_pieces(rows[i], few)), P.part_slots - kDownParts);
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
    float acc[NV], m_run = kAttnLowest, l_run = 0.f;
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
        const float corr = __builtin_amdgcn_exp2f(m_run - mn), p = __builtin_amdgcn_exp2f(sc - mn);
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
    // lanes -> wavefront (a wavefront without rows leaves (0, kAttnLowest, 0)) -> workgroup
    {
        const float mw = wave_max(m_run);
        const float fl = __builtin_amdgcn_exp2f(m_run - mw);
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
    for (int w = 1; w < NW; ++w) M = fmaxf(M, wm[w]);
#pragma unroll
    for (int e = 0; e < NE; ++e) O[e] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float ew = __builtin_amdgcn_exp2f(wm[w] - M);
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
    M = kAttnLowest; L = 0.f;
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
                const float c0 = __builtin_amdgcn_exp2f(M - mn), c1 = __builtin_amdgcn_exp2f(mj[j] - mn);
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

AttnPlan plan_attention_batched(const Dims &dm, int nb, int first)
{
    const bool stream = first < 0;
    const int H = dm.H, spare = stream ? kAttnSpareGroups / H : max(1, kAttnSharedGroups / (H * nb));
    // no sequence has more pieces than its longest context allows (64 / LPP positions a row, as in AttnShape); a group's is known
    const int row = dm.d >= 128 ? 16 : 32, most = attn_pieces(((stream ? dm.max_seq : first + nb) + row - 1) / row, nb <= kAttnFew);
    AttnPlan A;
    A.pieces = stream ? 1 + spare : spare;
    A.attn = (stream ? min(nb + spare, nb * most) : nb * min(spare, most)) * H;
    A.downs = stream ? down_parts_of(dm.h, dm.f, nb == 1) : down_parts_beside(dm.h, dm.f, nb == 1, A.attn, first);
    return A;
}

hipError_t launch_attention_batched(const StepParams &P, int nb, int first, const __half *w, const __half *kv, int *downs, hipStream_t s)
{
    const bool stream = P.attn_bstep != 0;
    if (nb < 1 || nb > kAttnBatchMax || (!stream && (first < 0 || first + nb > P.dm.max_seq))) return hipErrorInvalidValue;
    const AttnPlan plan = plan_attention_batched(P.dm, nb, stream ? -1 : first);
    const int spare = plan.pieces - (stream ? 1 : 0);
    const bool few = nb <= kAttnFew;
    DownPlan down;
    down.w = w;
    down.first = plan.attn;
    down.parts = plan.downs;
    *downs = down.parts;
    const dim3 grid(down.first + P.dm.h / (nb == 1 ? kDownRowsOne : kDownRows) * down.parts), block(kAttnBatchThreads);
    static_assert(down_lds<true>() <= 64 * 1024 && down_lds<false>() <= 64 * 1024, "the default limit");
    if (P.part_slots <= kDownParts) return hipErrorInvalidValue;
    switch (P.dm.d) {
#define CFPP_ATTN(D) \
    case D: \
        if (stream && nb == 1) hipLaunchKernelGGL((k_attention_batched<D, true, true>), grid, block, down_lds<true>(), s, P, nb, spare, few, kv, down); \
        else if (stream) hipLaunchKernelGGL((k_attention_batched<D, true, false>), grid, block, down_lds<false>(), s, P, nb, spare, few, kv, down); \
        else if (nb == 1) hipLaunchKernelGGL((k_attention_batched<D, false, true>), grid, block, down_lds<true>(), s, P, nb, spare, few, kv, down); \
        else hipLaunchKernelGGL((k_attention_batched<D, false, false>), grid, block, down_lds<false>(), s, P, nb, spare, few, kv, down); \
        break;
    CFPP_ATTN(64)
    CFPP_ATTN(80)
    CFPP_ATTN(128)
#undef CFPP_ATTN
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cfpp
