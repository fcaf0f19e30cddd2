/*
 * razer_tune.h -- launch-shape tuning hooks of the gfx950 RaZeR library.
 *
 * The paper's weight-only kernel is tuned offline: every matrix size is profiled ahead of time and the
 * number of SMs to launch is then picked per batch size when the kernel runs (Sec. 4.3; App. E, Tab. 13:
 * fewer, larger partitions cut the reduction stages of small problems).  The counterpart here: for a
 * problem (kernel family, activation rows m, weight rows, cols) the dispatch of razer_linear /
 * razer_linear_grouped takes its launch shape -- rows per workgroup, waves per K range, K-slices, which
 * of two kernels -- from a table compiled into the library (csrc/razer_tuned.inc), written by the
 * committed sweep `python -m paper_2501_04052_amd.tune` on the GPU; shapes that are not in the table
 * take a heuristic.  An entry chooses among the shapes of its family; which kernel serves a call is the
 * dispatch's own rule, and where that is the small-batch kernel at 2 .. 4 or 33 .. 128 rows, entries of
 * RAZER_TUNE_GEMV_QUAD and RAZER_TUNE_GEMM_SLICES have no effect on the launch (a forced shape of those
 * families keeps the call on its family's kernel).  Results never depend on the shape beyond fp32
 * summation order.
 *
 * Families and their parameters p[0..3] (unused ones 0):
 *   RAZER_TUNE_GEMV         m = 1 (and 2 .. 4 with rows longer than 32768 elements): p[0] = groups of 2 rows
 *                           per set of waves (2, 4 or 8), p[1] = sets of waves per workgroup (1 or 2; 2 only
 *                           with p[0] = 2)
 *   RAZER_TUNE_GEMV_QUAD    m = 2 .. 4, every block size and weight format: p[0] = groups of 4 rows per
 *                           workgroup (4 or 8)
 *   RAZER_TUNE_SMALL_BATCH  5 <= m where the small-batch kernel serves the call: p[0] = 2, p[1] = groups of 16
 *                           rows per workgroup (1, 2, 3, 4, 6; above 32 rows at most 4, FP16-scale format 3),
 *                           p[2] = waves that share K (8, or 16 with one group and at most 8 rows, 9 .. 16 rows
 *                           of 4096 elements or more, above 32 rows of 10240 or more, but not where K ends with half
 *                           a line of activations and the kernel takes whole steps; 0: the heuristic's number, when
 *                           forced 8; fewer where K has fewer steps of 128 elements; with 16, or with 0 in an entry,
 *                           4 above 32 rows where the workgroups outnumber the compute units).
 *                           The number of waves is the order of the sum over K.
 *                           p[0] = 0 or 1 (5 <= m <= 32) names a shape of the kernels this one replaced: an entry
 *                           selects only the size razer_workspace_bytes reports, forced it also asks for 8 waves:
 *                           p[0] = 0: fp32 K-slices of p[1] = 4 or 8 steps of 128 elements (p[2] = 1, 2, 4);
 *                           p[0] = 1 (m <= 16): none (p[1] = 1, 2; p[2] = 1, 2, 3, 4, 8; 8 only with p[1] = 2)
 *   RAZER_TUNE_GEMM_SLICES  33 <= m <= 128: p[0] = K-slices of the register-decode kernel (1 .. 16; forced, also
 *                           where the small-batch kernel would serve; above 128 rows only that)
 * For razer_linear_grouped `rows` is the sum over the group.  A shape the kernels are not built for is
 * ignored (the heuristic applies).  Every family, forced only: p[0] = -1: the heuristic, as if neither a
 * shape were forced nor one on record.
 */
#ifndef RAZER_TUNE_H
#define RAZER_TUNE_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

enum { RAZER_TUNE_GEMV = 0, RAZER_TUNE_GEMV_QUAD = 1, RAZER_TUNE_SMALL_BATCH = 2, RAZER_TUNE_GEMM_SLICES = 3,
       RAZER_TUNE_FAMILIES = 4 };

/* For the tuner: while set, every dispatch of `family` made by THIS host thread uses p[0..3] (HOST
 * array) instead of the table -- also razer_workspace_bytes, so size the workspace after forcing.
 * p = NULL clears the family's override; family = -1 with p = NULL clears all.  Returns 0, or 2 for a
 * bad family. */
int razer_tune_force(int family, const int32_t *p);

/* The shape on record for a call of that family: copies it to p[0..3] (HOST) and returns 1 if it is this
 * thread's forced shape, 2 if it comes from the built-in table; returns 0 (p untouched) when the heuristic
 * applies.  (It does not say which kernel serves the call.) */
int razer_tune_lookup(int family, int64_t m, int64_t rows, int64_t cols, int32_t *p);

/* Number of entries of the built-in table. */
int razer_tune_table_size(void);

#ifdef __cplusplus
}
#endif
#endif /* RAZER_TUNE_H */
