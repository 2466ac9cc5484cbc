/*
 * cfpp profiling and test aids - NOT part of the library's ABI.
 *
 * These declarations exist only in the profiling build of the library
 * (libcfpp_profile.so, the same sources compiled with -DCFPP_PROFILE); the
 * product library (libcfpp.so) exports none of them, its kernels carry no
 * tracer and honour no skip bits.  They may change at any time.  Callers:
 * the kernel-timeline and counter-calibration runs behind the figures in the
 * design notes, and the tests that compare a block's intermediates with the CPU
 * oracle's.
 */
#ifndef CFPP_PROFILE_H
#define CFPP_PROFILE_H

#include "cfpp.h"

#ifdef __cplusplus
extern "C" {
#endif

/* cfpp_set_option(): profiling switches.
 * CFPP_OPT_PROFILE_SKIP  Bits 0-3: sub-steps to skip so that the others can be
 *                        timed alone (results are then wrong).  Bit 4 (16):
 *                        workgroup ((value >> 8) & 0xfff) records a per-wavefront
 *                        timeline (mode 2: of layer ((value >> 20) & 255) - 1, of
 *                        the last layer when those bits are 0); bit 5 (32): every
 *                        workgroup records a few time stamps of the last layer
 *                        (mode 2); both are read back with cfpp_debug_read(which
 *                        = 4) and leave the results intact.
 * CFPP_OPT_EPOCH_LIMIT   number of tagged-word epochs after which the library
 *                        re-zeroes the epoch counter (default 0xF0000000); a test
 *                        sets it to a few launches' worth to exercise that path. */
#define CFPP_OPT_PROFILE_SKIP 100
#define CFPP_OPT_EPOCH_LIMIT  101

/* Test tap: synchronises `stream`, then copies a workspace intermediate of the
 * most recent block to HOST memory as fp32.  which: 0 = rotated q [batch, h],
 * 1 = GELU(up) [batch, f], 2 = down projection incl. bias [batch, h] (launch
 * modes 0 and 1; mode 2 keeps it in registers), 3 = attention output before the
 * output projection [batch, h] (modes 0 and 1), 4 = raw timeline words.
 * count = number of floats to copy (from the start). */
cfpp_status cfpp_debug_read(cfpp_ctx *ctx, int32_t which, float *dst_host, size_t count,
                            cfpp_stream stream);

/* The plan of one pass of cfpp_stack_prefill_gemm over n_tokens <= rows tokens (host
 * arithmetic, no GPU) in its tiled products, before passes of up to 64 tokens take the
 * narrow ones (cfpp_debug_prefill_narrow) and passes of 65 .. 1024 tokens other tiles
 * (cfpp_debug_prefill_tiles).  plan[0..3]: the first product (QKV, MLP-up), plan[4..7]: the
 * second (output projection, MLP-down); of each the tokens, output features and K
 * values of a tile's step and the parts K is split into.  past[0..3]: by how many rows
 * the tiles' loads reach past the activations and the weights of the first product,
 * then of the second: 0 unless something is wrong. */
cfpp_status cfpp_debug_prefill_plan(const cfpp_config *cfg, int32_t rows, int32_t n_tokens,
                                    int32_t plan[8], int32_t past[4]);

/* The same with the tiles that a pass of 65 .. 1024 tokens takes; the first product of more than 512 tokens:
 * cfpp_debug_prefill_long. */
cfpp_status cfpp_debug_prefill_tiles(const cfpp_config *cfg, int32_t rows, int32_t n_tokens,
                                     int32_t plan[8], int32_t past[4]);

/* What the first product of a pass of more than 512 tokens runs as, behind the two above (the second product is theirs).
 * plan[0..1]: tokens and output features of its tile, plan[2]: MLP-up rows that the launch takes (all of them: there
 * is no other), plan[3..4]: the tile of the launch that takes the others, or 0.  past[0..1]: by how many rows the tiles'
 * loads reach past the weights in the first launch, in the second. */
cfpp_status cfpp_debug_prefill_long(const cfpp_config *cfg, int32_t rows, int32_t n_tokens,
                                    int32_t plan[5], int32_t past[2]);

/* The narrow products of a pass of n_tokens tokens on a device of n_cu CUs (host arithmetic, no
 * GPU): plan[0] 1 if the pass takes them; plan[1], plan[2] rows and tiles of a workgroup of the
 * first product, plan[3], plan[4] of the second (of the output projection alone where MLP-down
 * runs beside the attention), plan[5] the parts of its K, plan[6] the sets of tokens. */
cfpp_status cfpp_debug_prefill_narrow(const cfpp_config *cfg, int32_t rows, int32_t n_tokens, int32_t n_cu, int32_t plan[7]);

/* The same for tokens from position pos0 on, in a scratch whose last part, for the parts of products and of the attention, has part_bytes
 * bytes (0: what it has).  plan[0] as above; plan[1] parts of MLP-down beside the attention, 0: behind it; plan[2] parts of the
 * second product's K (as plan[5] above); plan[3] parts of the attention's keys; plan[4] workgroups of MLP-down.  Where the pass does not take
 * the narrow products, plan[1] is 1 if what was planned before is as it was. */
cfpp_status cfpp_debug_prefill_beside(const cfpp_config *cfg, int32_t rows, int32_t n_tokens, int32_t pos0, int32_t n_cu,
                                      size_t part_bytes, int32_t plan[5]);

/* The attention of the batched path (host arithmetic, no GPU) with n sequences' step (first < 0; 1 for one sequence) or
 * n tokens of a prompt's group from position first on: plan[0] 1 if the group attends together; plan[1] pieces of a head, at most; plan[2]
 * workgroups ahead of MLP-down's; plan[3] parts of MLP-down, plan[4] its workgroups. */
cfpp_status cfpp_debug_attention_plan(const cfpp_config *cfg, int32_t n, int32_t first, int32_t plan[5]);

/* Where cfpp_stack_prefill_gemm keeps a layer's intermediates in the caller's scratch, byte
 * offsets: at[0], at[1] gamma_1 x and gamma_2 x, at[3] the attention output, at[4] GELU(up),
 * each as rows of groups of 32 fp16 heads and then their 32 fp16 remainders (value = head +
 * remainder; after a pass through the narrow products in another order), halves[0] fp16 values from row to row (at[4]: halves[1]); at[2] the rotated
 * queries, fp32 [rows][hidden].  After the call they are the last layer's, where the
 * second product's K is in one part (cfpp_debug_prefill_plan); its parts overwrite the queries. */
cfpp_status cfpp_debug_prefill_scratch(const cfpp_config *cfg, int32_t rows, size_t at[5], int32_t halves[2]);

/* GELU of n fp32 values z (DEVICE) as the prompt-sized kernels' epilogues work it out
 * and as the other kernels do, with the device library's erff or tanhf (flags:
 * CFPP_FLAG_TANH_GELU or 0), into two DEVICE arrays. */
cfpp_status cfpp_debug_gelu(const float *z, float *epilogue, float *library, int32_t n, int32_t flags,
                            cfpp_stream stream);

/* Plain streaming kernels whose HBM traffic is known exactly, used to find the
 * streaming bandwidth this GPU sustains and to scale hardware traffic counters.
 * cfpp_stream_read loads every 16-byte word of src (DEVICE, `bytes` a multiple of
 * 16) once and XORs a checksum into sink (DEVICE, uint32[grid], caller-zeroed);
 * cfpp_stream_copy copies src to dst.  grid <= 65536, threads 256 or 512,
 * unroll = 16-byte loads in flight per thread (2, 4 or 8). */
cfpp_status cfpp_stream_read(const void *src, size_t bytes, void *sink, int32_t grid,
                             int32_t threads, int32_t unroll, cfpp_stream stream);
cfpp_status cfpp_stream_copy(const void *src, void *dst, size_t bytes, int32_t grid,
                             int32_t threads, cfpp_stream stream);

#ifdef __cplusplus
}
#endif
#endif /* CFPP_PROFILE_H */
