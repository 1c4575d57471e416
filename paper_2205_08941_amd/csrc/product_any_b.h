// LDS-ring product kernels for the orbital counts without tuned kernels of their own
// (5 <= b <= 16, b != 9), FP64 and FP32 operands.
#pragma once

#include "bsm_internal.h"

namespace bsm {

// Rows per tile of these kernels: up to b = 8 the sums of 8 rows leave room for two
// waves per SIMD, above that the sums of 4 do; products of few tiles take 2 (the line of
// product.hip's ring_rows).
inline int any_b_rows(int b, bool few) { return few ? 2 : b <= 8 ? 8 : 4; }
inline bool any_b_ring(int b) { return b >= 5 && b <= 16 && b != 9; }

// One launch over a one-wave ring plan (variant 4) of any_b_rows rows, direct or
// transposed; operands must fit buffer resources (fits_buffers).
void launch_any_b(hipStream_t st, const Plan *plan, const double *A, const double *B, double *C, double alpha,
                  double beta, const double *zblk, int64_t a_bytes, int64_t b_bytes);
void launch_any_b(hipStream_t st, const Plan *plan, const float *A, const float *B, double *C, double alpha,
                  double beta, const float *zblk, int64_t a_bytes, int64_t b_bytes);
// Whether FP64 operands of these patterns fit buffer resources.
bool fits_buffers(const bsm_pattern_s *PA, const bsm_pattern_s *PB);

}  // namespace bsm
