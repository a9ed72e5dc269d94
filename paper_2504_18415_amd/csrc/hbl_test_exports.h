/*
 * Exports of libhbitlinear.so that exist for the test suite only.  They are not part of the public
 * interface (include/hbitlinear.h) and may change with the kernels they look into.
 */
#ifndef HBL_TEST_EXPORTS_H
#define HBL_TEST_EXPORTS_H

#include "hbitlinear.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Host only (no launch, no device access): the GEMM launch a grouped call would make for these problems (every T in
 * 1..64, one bit width, n_problems <= 8; only T, K, N, bits and hadamard are read).
 *   route             1: weight streaming   2: mid-size (as in hbl_test_forward_route)
 *   ksplit[i]         weight streaming: K slices per 32-row weight tile of problem i (inside a workgroup when every
 *                     T <= 16, over workgroups otherwise - the last of them to finish adds the slices); else 0
 *   gemm_workgroups   weight streaming: grid size; else 0
 *   arrival_counters  groups of four row tiles whose K range is split over workgroups (0 = none)
 */
int hbl_test_grouped_plan(const hbl_problem* problems, int n_problems, int* route, int* ksplit, int* gemm_workgroups,
                          int* arrival_counters);

/*
 * Host only: the kernel that a single forward call of this shape ends in, as the dispatch picks it (norm != 0: with the
 * RMS normalisation).  0: one launch for quantiser and product   1: weight streaming   2: mid-size   3: prefill
 * 4: one launch for short rows; or a negative status.
 */
int hbl_test_forward_route(int64_t T, int64_t K, int64_t N, int x_dtype, int bits, int hadamard, int norm);

/*
 * Host only: the tile (numbers below; 4: 128 features x 32 or 64 tokens) that the GEMM on codes of this form takes, in the
 * stage-level calls and in forward calls that end in the mid-size (3) or a prefill kernel; or a negative status.
 */
int hbl_test_gemm_tile(int64_t T, int64_t K, int64_t N, int code_form);

/*
 * The integer contraction of Eq. 7 through one named workgroup tile of a prefill GEMM kernel (T > 64):
 * acc[t][o] = sum_k q[t][k] c[o][k] as int32 [T, N], on a shape of the caller's choice - the forward
 * calls pick the tile from the shape, so most tiles would otherwise be reachable at benchmark sizes only.
 *   code_form  HBL_CODES_INT8 (int8 matrix-core kernel, codes [T, K] bytes) or HBL_CODES_BF6 (fp6 x fp4
 *              kernel, code records; K >= 512)
 *   tile       0: 256 x 256   1: 128 x 128   2: 512 features x 128 tokens
 *              3: the mid-size kernel, K cut over the waves of a workgroup (HBL_CODES_BF6 only)
 *              10: 256 features x 128 tokens   11: 128 x 128, two stages   12, 13: 192 features x 128 tokens, two and four
 *              stages (11 to 13: HBL_CODES_BF6 only)
 */
int hbl_test_gemm_i32_tile(const void* codes, int code_form, int64_t T, int64_t K, const void* Wq_packed,
                           int64_t N, int32_t* acc, int tile, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* HBL_TEST_EXPORTS_H */
