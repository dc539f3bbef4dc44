/*
 * Entry points of the same library that serve its benchmarks and tests, not its users: measured
 * ceilings of the device and hooks that pin a kernel configuration.  Nothing in the linear-layer
 * path depends on them.  Conventions (device pointers, status codes, streams) as in fp6.h.
 */
#ifndef FP6_BENCH_H
#define FP6_BENCH_H

#include "fp6.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Diagnostics for benchmarks: empirical ceilings of the device, measured with the request
 * patterns of the linear kernels (the paper's Section 7.1 reads the same two utilisations
 * off its profiler: DRAM bandwidth and Tensor-Core use).
 *   fp6_probe_read: `buffer` (device) is cut into pieces of 8 KB; 1024 waves sweep it front to
 *     back, wave w reading pieces w, 1024 + w, 2048 + w, ... with the non-temporal 128-bit loads
 *     of the weight path, sixteen in flight, and XOR the 32-bit words of their pieces together
 *     into sink[w] (device, 1024 x uint32).  fp6_probe_read_bytes(bytes) is the number of bytes
 *     actually read (a whole, even number of pieces per wave).  bytes >= 16 MiB, else FP6_ERR_SHAPE.
 *   fp6_probe_mfma: 4096 waves (four per SIMD) each issue iters x 4 independent
 *     v_mfma_f32_32x32x16_f16 (32768 flop each) on register operands; `sink` (device,
 *     fp6_probe_mfma_sink_bytes() bytes) receives one float per lane.
 */
fp6_status fp6_probe_read(const void *buffer, size_t bytes, void *sink, void *stream);
size_t fp6_probe_read_bytes(size_t bytes);
fp6_status fp6_probe_mfma(int64_t iters, void *sink, void *stream);
size_t fp6_probe_mfma_sink_bytes(void);

/*
 * Tuning hook for benchmarks and tests: force the split-K factor used by fp6_linear, fp5_linear,
 * fp4_linear, fp3_linear and fp16_linear (0 = choose automatically, the default).  Process-wide; affects the
 * workspace size queries as well.  Values the shape cannot honour are clamped.
 */
void fp6_tuning_set_split_k(int split_k);

/*
 * Tuning hook for benchmarks and tests: force the block tile of the kernel used for N > 64:
 * block_rows in {128, 256} output channels x block_tokens in {64, 128} tokens, or 256 x 256; any
 * other pair restores the automatic choice.  Where a weight format lacks a shape the next smaller one
 * is used (fp16_linear and 64 tokens: 128 rows; group scales: 256 x 128 and 128 x 64).
 * Process-wide; affects the workspace size queries as well.
 */
void fp6_tuning_set_tile(int block_rows, int block_tokens);

/*
 * What a call would launch for the tokens around `token` (a call whose activations exceed 2 GiB is cut into launches
 * that are planned one by one), under the tuning hooks in force, given a workspace of workspace_bytes (refused with
 * FP6_ERR_WORKSPACE like the call).  Host arithmetic only.  weight_bits: 6, 5, 4, 3, -6 (fp6g_linear) or 16 (fp16_linear).
 */
enum { FP6_KERNEL_STREAM = 0, FP6_KERNEL_TILED = 1, FP6_KERNEL_BLOCK = 2 };
typedef struct {
    int kernel;                    /* FP6_KERNEL_* */
    int block_rows, block_tokens;  /* output piece of a workgroup */
    int split_k;                   /* k slices */
    int64_t first_token, tokens;   /* of the launch */
    size_t counter_bytes;          /* arrival counters, at the start of the workspace (0 without k slices) */
    size_t partial_offset;         /* where its partial sums start ... */
    size_t partial_bytes;          /* ... and the room for them that the call asks for (0 without k slices) */
} fp6_launch_plan;
fp6_status fp6_tuning_plan(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes,
                           fp6_launch_plan *plan);
/* Groups of k-tiles of a workgroup of that launch (waves that share an output piece and meet in LDS); 0 where it is refused. */
int fp6_tuning_plan_k_groups(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes);
/*
 * Partial sums of that launch, bytes behind the counters: `used` by it (0 without k slices), and `required` of the workspace, without
 * which the call is refused or launches something else.  More is required than used where the block that is launched takes fewer
 * k slices than the one that the size query is made for (then also by a launch without any).
 */
fp6_status fp6_tuning_plan_partials(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes, size_t *used,
                                    size_t *required);

/*
 * quantize_pack calls with a scale per row (weight_bits 6, 5, 4, 3) read W in one launch where that is faster:
 *   fp6_tuning_pack_parts: blocks that a row tile is divided among in that launch (1: they exchange nothing); 0: two
 *     launches; -1: the shape or the width is refused.  Host arithmetic only.
 *   fp6_tuning_set_pack_polls: how often a block looks for the other parts of its row tile before it reads their columns itself
 *     (0: not once; negative: the default).  Process-wide.  The packed bytes do not depend on it.
 */
int fp6_tuning_pack_parts(int weight_bits, int64_t M, int64_t K);
void fp6_tuning_set_pack_polls(int polls);

#ifdef __cplusplus
}
#endif

#endif /* FP6_BENCH_H */
