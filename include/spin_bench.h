/*
 * spin_bench.h -- measurement aids of the library declared in spin.h.  Nothing
 * here is part of the protocol: per-kernel HIP-event timing that benchmarks
 * switch on around a timed region, and a register-only int8 MFMA loop that
 * measures what the matrix cores sustain on given operand bytes.  Conventions
 * (device pointers, streams, return codes) as in spin.h.
 */
#ifndef SPIN_BENCH_H
#define SPIN_BENCH_H

#include "spin.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Per-kernel timing for benchmarks.  While enabled, every kernel the library
 * launches is bracketed by a pair of HIP events recorded on the caller's
 * stream; the events are created on demand, so while (and only while) timing
 * is enabled the library's calls do allocate event objects.  A launch on a
 * stream that is being captured into a HIP graph is not timed (recorded events
 * of a capture cannot be read), whatever the switch says.
 * spin_profile_read waits for the recorded events and returns the summed
 * duration in milliseconds and the number of launches of one kernel class
 * since the last spin_profile_reset.  The record is process-wide and guarded
 * by a mutex; spin_profile_reset must not run while another thread's timed
 * launches are still being enqueued. */
typedef enum {
    SPIN_KERNEL_RANDOM = 0,
    SPIN_KERNEL_SHARE = 1,
    SPIN_KERNEL_OPEN = 2,
    SPIN_KERNEL_BEAVER_MUL = 3,
    SPIN_KERNEL_TRUNC = 4,
    SPIN_KERNEL_PACK = 5,       /* open + digit split + fragment layout for the limb GEMM */
    SPIN_KERNEL_GEMM_LIMB = 6,
    SPIN_KERNEL_GEMM_VALU = 7,
    SPIN_KERNEL_LINCOMB = 8,    /* lincomb_trunc, completed_square_trunc */
    SPIN_KERNEL_BINARY = 9,     /* bshare, bopen, beaver_and */
    SPIN_KERNEL_CAST = 10,      /* spin_cast_64_to_32 */
    SPIN_KERNEL_PROBE = 11,     /* spin_probe_mfma */
    SPIN_KERNEL_MUL_TRUNC = 12, /* spin_beaver_mul_trunc */
    SPIN_KERNEL_GEMM_RESIDUE = 13,   /* residue GEMM; its packs count as SPIN_KERNEL_PACK */
    SPIN_KERNEL_COMBINE = 14,        /* residues back to ring words */
    SPIN_KERNEL_GEMM_DIRECT = 15,    /* small matmuls in one launch */
    SPIN_KERNEL_COUNT = 16
} spin_kernel;
void spin_profile_enable(int on);
spin_status spin_profile_read(int kernel, double *total_ms, unsigned *launches);
void spin_profile_reset(void);

/* Measurement aid: the int8 matrix-core rate the chip sustains on given operand bytes.  Every wave
 * of `blocks` workgroups (4 waves each) loads 24 MFMA operand fragments of 1 KiB from `operands`
 * ([24][128] uint64_t: 16 left fragments for two 32x32 tiles, then 8 right fragments; lane l of a wave
 * reads bytes 16 l .. 16 l + 15 of each) and issues, `iters` times, the 72 v_mfma_i32_32x32x32_i8 of one
 * k-step of the 64-bit limb GEMM (digit pairs i + j <= 7, pairs of one diagonal sharing an
 * accumulator), with no memory or LDS access inside the loop: blocks * 4 * iters * 72 * 65536 int8
 * operations per call.  sink[blocks * 256] receives each thread's wrapped int32 sum of its
 * accumulator registers, sign-extended (it keeps the loop alive and lets a test check the
 * arithmetic).  1 <= blocks <= 2^20, 1 <= iters <= 2^20.  Time it with spin_profile_* or events.  */
spin_status spin_probe_mfma(const uint64_t *operands, int blocks, int iters, uint64_t *sink,
                            spin_stream stream);

/* The kernel that a matmul on the digit path (SPIN_GEMM_LIMB_MFMA) takes, and a matmul by a kernel that the caller names.  The calls of
 * spin.h choose by estimated time; these two let a test or a measurement say what it runs, and leave the choice alone.
 * parts: workgroups that share an output tile, 1 to 16 (tile kernels; 1 for the others). */
typedef enum {
    SPIN_WAY_DIRECT = 0,        /* one launch on the vector ALU */
    SPIN_WAY_ROWS = 1,          /* row kernel: 64-bit words, at most three parties, K <= 16352 */
    SPIN_WAY_FULL_TILES = 2,    /* tiles of 128 x 64 (64-bit words), 128 x 128 (32-bit) */
    SPIN_WAY_HALF_TILES = 3,    /* 64 x 64, 64 x 128 */
    SPIN_WAY_QUARTER_TILES = 4, /* 32-bit words: 64 x 64 */
    SPIN_WAY_RESIDUES = 5,      /* residue GEMM, by the best plan for the workspace: 64-bit words */
    SPIN_WAY_SEPARATE = 6       /* of a grouped call: one product after another */
} spin_way_kernel;
typedef struct { int kernel; int parts; } spin_matmul_way;

/* What the library would take for a product of 32- or 64-bit words if its digit kernels and the direct one were all there are (the residue
 * GEMM and the recursion over Z_2^32, where they are estimated to be faster, come before), and for the products of a grouped
 * call.  Launches nothing and touches no pointer of desc. */
spin_status spin_matmul_way_of(int word_bits, int n, int batch, int M, int N, int K, spin_matmul_way *way);
spin_status spin_matmul_grouped_way_of(int n, int groups, const spin_matmul_group *desc, spin_matmul_way *way);

/* spin_beaver_matmul (word_bits 64; spin_beaver_matmul_nt with y_transposed), spin32_beaver_matmul (32) and
 * spin_beaver_matmul_grouped on the path SPIN_GEMM_LIMB_MFMA, with their arguments and workspaces, by `way` (not
 * SPIN_WAY_SEPARATE, nor SPIN_WAY_DIRECT for a grouped call).  SPIN_EINVAL: not a product of that kernel, or not so many parts of whole pairs of k-steps;
 * SPIN_EWORKSPACE too where no plan of the residue GEMM fits; SPIN_ERANGE: not in one launch. */
spin_status spin_matmul_by(spin_matmul_way way, int word_bits, int n, int batch, int M, int N, int K, const void *X, const void *Y,
                           const void *A, const void *B, const void *C, void *Z, int y_transposed, void *workspace,
                           size_t workspace_bytes, spin_stream stream);
spin_status spin_matmul_grouped_by(spin_matmul_way way, int n, int groups, const spin_matmul_group *desc, void *workspace,
                                   size_t workspace_bytes, spin_stream stream);

#ifdef __cplusplus
}
#endif
#endif /* SPIN_BENCH_H */
