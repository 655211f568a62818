// Norms that do more in their launches, and column sums that share theirs (norm.hip).
#pragma once
#include "common.h"

namespace tmk {

// tm_op_norm_fwd; copy (or NULL): x as it is, 16-byte aligned, no part of it x or out
int norm_fwd_and_copy(int dtype, int kind, int64_t T, int64_t h, double eps, const void *x, const void *gain, const void *offset,
                      void *out, float *mean, float *rstd, void *copy, hipStream_t s);

struct ColumnSum {  // out[c] (+)= the sum over the rows of dy [T][n]; dy starts on 16 bytes, n is a multiple of 8
  const void *dy;
  float *out;
  int64_t n;
};

// bytes of partial_sums for `width` columns in all (0: few rows need none)
int64_t column_sums_scratch_bytes(int64_t T, int64_t width);

// tm_op_norm_bwd or, with dx_colsum, tm_op_norm_bwd_colsum; and up to three column sums (tm_op_bias_grad, the same bits)
// whose launches they share with the norm's own: they are read behind its first launch, so that no dy of theirs may overlap dx.
// partial_sums: not the norm's scratch.
int norm_bwd_and_column_sums(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean,
                             const float *rstd, const void *gain, const void *dres, void *dx, float *dgain, float *doffset,
                             float *dx_colsum, void *scratch, const ColumnSum *sums, int count, void *partial_sums,
                             int accumulate, hipStream_t s);

}  // namespace tmk
