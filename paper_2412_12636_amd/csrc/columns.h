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

// A norm's backward pass whose partial rows have not been added up yet.
struct NormSums {
  const float *partial = nullptr;  // NULL: none
  int rows;
  int64_t h;
  float *out[3];
};
// bytes of a norm's partial rows
int64_t norm_bwd_partial_bytes(int dtype, int64_t T, int64_t h);
// tm_op_norm_bwd or, with dx_colsum, tm_op_norm_bwd_colsum, up to its partial rows (in scratch): *later adds them up as the
// `earlier` of the next function
int norm_bwd_rows(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean, const float *rstd,
                  const void *gain, const void *dres, void *dx, float *dgain, float *doffset, float *dx_colsum, void *scratch,
                  NormSums *later, hipStream_t s);

// tm_op_norm_bwd or, with dx_colsum, tm_op_norm_bwd_colsum; and up to three column sums (tm_op_bias_grad, the same bits)
// whose launches they share with the norm's own: they are read behind its first launch, so that no dy of theirs may overlap dx.
// partial_sums: not the norm's scratch, and neither holds the partial rows of `earlier`, which the same launch adds up.
int norm_bwd_and_column_sums(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean,
                             const float *rstd, const void *gain, const void *dres, void *dx, float *dgain, float *doffset,
                             float *dx_colsum, void *scratch, const ColumnSum *sums, int count, void *partial_sums,
                             const NormSums &earlier, int accumulate, hipStream_t s);

}  // namespace tmk
