/* hexa_moe_bench.h -- measurement helpers of libhexa_moe.  NOT part of the layer's interface
 * (include/hexa_moe.h): bench.py uses them to time the library's kernels one by one and to
 * measure the matrix rate the part sustains.  They live in the same shared library because they
 * have to bracket the library's own launches. */
#ifndef HEXA_MOE_BENCH_H
#define HEXA_MOE_BENCH_H

#include "hexa_moe.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Per-kernel timing.  While enabled, every kernel the library launches is bracketed by two HIP
 * events on its stream; enabling (or disabling) discards earlier records.  This is the only part
 * of the library that creates HIP objects, so it must stay off under stream capture.
 * hexa_moe_profile_read(i, ...) waits for the recorded events and returns the i-th distinct
 * kernel label with its summed duration in ms and its launch count; returns 0 once i is past
 * the last label (or on a HIP error), else 1.  The record list is guarded by a mutex; the
 * recording state is process-wide. */
HEXA_API void hexa_moe_profile_enable(int on);
HEXA_API int hexa_moe_profile_read(int i, const char **label, float *ms_total, int *launches);

/* Enqueues a register-only bf16 MFMA loop: `workgroups` workgroups of four wavefronts, each wavefront
 * issuing iters * 32 16x16x32 MFMAs (variant 2: iters * 16 32x32x16 MFMAs; the same FLOP), and writes
 * the FLOP count of the launch to *flop (host).  Timed by the caller on `stream`, it gives the matrix
 * rate the part sustains under its power limit, which depends on the operand bits:
 *   variant 0  16x16x32, pseudo-random operands of the layer's magnitude (what bench.py reports)
 *   variant 1  16x16x32, all-zero operands
 *   variant 2  32x32x16, pseudo-random operands
 * sink: dev, >= 4 bytes, never written in practice. */
HEXA_API hexa_status hexa_moe_mfma_probe(int32_t variant, int32_t workgroups, int32_t iters, float *sink,
                                void *stream, double *flop);

/* How the launches of a shape are cut (host only; depends on the shape alone).  Tests use it to see that a
 * shape takes the kernels they are about. */
typedef struct {
    int32_t fc1_tile, fc2_tile, bwd_fc2_tile, bwd_fc1_tile; /* rows and columns of an output tile of each
                                  contraction launch (bwd_fc2 / bwd_fc1: both contractions of the layer) */
    int32_t fc2_shares;        /* shares of K in which FC2 runs (1: unsplit) */
    int32_t chunk_rows;        /* rows per chunk that the token contractions aim at */
    int64_t partial_buffers;   /* partial weight gradients the workspace has room for, per weight matrix */
    int64_t index_chunk_ids, index_chunks;   /* index build: ids per workgroup, workgroups */
    int64_t prologue_blocks;   /* workgroups of the backward prologue (with dgate) */
    int32_t wide;              /* fp32: bit i set where launch i (in the order of the tiles) takes tiles of 128 rows and 64 columns */
    int32_t thin;              /* 16 bits: bits 0, 1 set where fc1, fc2 take tiles of 32 rows and 128 columns (few rows) */
} hexa_moe_plan;
HEXA_API hexa_status hexa_moe_launch_plan(const hexa_moe_shape *shape, hexa_moe_plan *plan);

#ifdef __cplusplus
}
#endif
#endif /* HEXA_MOE_BENCH_H */
