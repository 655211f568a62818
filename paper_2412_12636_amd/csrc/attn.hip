// Causal attention entry points: argument checks and dispatch between the MFMA flash-style
// kernels (bf16 and fp32, head sizes up to 128) and the plain-ALU kernels (everything else,
// tensors off the 16-byte alignment, and very short sequences of many walks).
#include "attn.h"
#include "../../include/tm_ops.h"

using namespace tmk;

static int check_attn(const char *what, int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  if (dtype != TM_DTYPE_FP32 && dtype != TM_DTYPE_BF16) return fail(TM_EINVAL, "%s: unknown dtype %d", what, dtype);
  if (seq <= 0 || batch <= 0 || nq <= 0 || nkv <= 0 || d <= 0) return fail(TM_EINVAL, "%s: empty shape", what);
  if (nq % nkv) return fail(TM_ESIZE, "%s: %lld query heads are not a multiple of %lld kv heads", what, (long long)nq, (long long)nkv);
  if (d % 8 || d > 256) return fail(TM_ESIZE, "%s: head size %lld must be a multiple of 8, at most 256", what, (long long)d);
  if (nq > 65535 || batch > 65535) return fail(TM_ESIZE, "%s: more than 65535 heads or batch entries", what);
  if (seq * batch * (nq + 2 * nkv) * d >= (1LL << 40)) return fail(TM_ESIZE, "%s: tensor too large", what);
  if (!(dtype == TM_DTYPE_BF16 && d == 128) && seq > attn_generic_max_seq())
    return fail(TM_ESIZE, "%s: sequences above %d need bf16 with head size 128", what, attn_generic_max_seq());
  return TM_OK;
}

// Very short sequences of many (entry, query head) walks stay with the kernels of one row per wave (but for bf16 with head
// size 128, which has no other kernel): a tile holds 32 or 64 positions, and what such a walk costs in tiles depends on their
// number, 1 for any of these lengths.  Up to how many positions that is the faster way, from both kernels' times at 1 to 24
// positions, 8 to 16384 walks, head sizes 8 to 128 (tiles / rows, us; fwd and bwd):
//   fp32, 16384 walks of 1 position, heads of 64: 205 / 23, 620 / 68; of 4: 209 / 120, 624 / 339; of 6: 209 / 177, 630 / 518;
//     of 8: 210 / 268, 634 / 1147; 8192 walks of 8, heads of 96: 219 / 178, 629 / 865; 256 walks of 4: 8.0 / 9.2, 24.0 / 21.9
//   bf16, 16384 walks of 1 position, heads of 64: 70 / 24, 180 / 79; of 2: 70 / 51, 183 / 199; of 3: 72 / 91, 189 / 277; heads
//     of 8: of 4: 57 / 35, 147 / 99; of 8: 58 / 78, 148 / 232; 1024 walks, heads of 64: rows are never the faster way
// Near a limit the two differ by 10 to 20 % either way.
static int row_kernel_positions(int dtype, bool bwd, int64_t walks, int64_t d) {
  if (dtype == TM_DTYPE_FP32) {
    if (d > 64) return walks >= 512 ? (bwd || d == 128 ? 6 : 8) : walks > (bwd ? 128 : 256) ? 4 : 0;
    if (walks >= 512) return d <= 8 ? 8 : d <= 16 || d > 32 ? 6 : walks >= 2048 ? 5 : 4;
    return d <= (bwd ? 8 : 16) ? 4 : 0;
  }
  if (walks >= 2048)
    return bwd ? (d <= 8 ? 4 : d <= 24 || d > 64 ? 3 : d <= 48 ? 2 : 1) : (d <= 8 ? 5 : d <= 16 ? 4 : d <= 32 ? 3 : 2);
  if (walks >= 512) return bwd ? (d <= 8 ? 3 : d <= 16 ? 2 : 0) : (d <= 8 ? 4 : d <= 16 ? 3 : d <= 24 ? 2 : 0);
  return !bwd && d <= 8 ? 4 : 0;
}
static bool rows_pay(int dtype, bool bwd, int64_t seq, int64_t walks, int64_t d) {
  return !(dtype == TM_DTYPE_BF16 && d == 128) && seq <= row_kernel_positions(dtype, bwd, walks, d);
}

// The tiles move 16 bytes at a time.  Tensors off that alignment go to the kernels of one row per wave, which read element by
// element (but for bf16 with head size 128, which has always had the tiles alone).
static bool tiles_take(int dtype, int64_t d, const void *a, const void *b) {
  return (dtype == TM_DTYPE_BF16 && d == 128) || !((((uintptr_t)a) | ((uintptr_t)b)) & 15);
}

extern "C" int tm_op_attn_fwd(int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d,
                              const void *qkv, void *ctx, float *lse, void *stream) {
  if (int e = check_attn("attn_fwd", dtype, seq, batch, nq, nkv, d)) return e;
  if (!qkv || !ctx || !lse) return fail(TM_EINVAL, "attn_fwd: NULL pointer");
  hipStream_t s = (hipStream_t)stream;
  if (rows_pay(dtype, false, seq, batch * nq, d) || !tiles_take(dtype, d, qkv, ctx))
    return attn_fwd_generic_launch(dtype, seq, batch, nq, nkv, d, qkv, ctx, lse, s);
  if (attn_mfma_supported(dtype, seq, batch, nq, nkv, d)) return attn_fwd_mfma_launch(seq, batch, nq, nkv, d, qkv, ctx, lse, s);
  if (attn_f32_supported(dtype, seq, batch, nq, nkv, d)) return attn_fwd_f32_launch(seq, batch, nq, nkv, d, qkv, ctx, lse, s);
  return attn_fwd_generic_launch(dtype, seq, batch, nq, nkv, d, qkv, ctx, lse, s);
}

extern "C" int64_t tm_op_attn_bwd_scratch_bytes(int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv,
                                                int64_t d) {
  if (int e = check_attn("attn_bwd_scratch_bytes", dtype, seq, batch, nq, nkv, d)) return e;
  const int64_t dvec = (batch * nq * seq + 63) / 64 * 64;  // the row statistics D, padded to 256 bytes
  const bool tiled = attn_mfma_supported(dtype, seq, batch, nq, nkv, d) || attn_f32_supported(dtype, seq, batch, nq, nkv, d);
  const int64_t part = tiled ? attn_bwd_mfma_partial_floats(seq, batch, nq, nkv, d) : 0;
  return (dvec + part) * (int64_t)sizeof(float);
}

extern "C" int tm_op_attn_bwd(int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d,
                              const void *qkv, const void *ctx, const void *dctx, const float *lse, void *scratch,
                              void *dqkv, void *stream) {
  if (int e = check_attn("attn_bwd", dtype, seq, batch, nq, nkv, d)) return e;
  if (!qkv || !ctx || !dctx || !lse || !scratch || !dqkv) return fail(TM_EINVAL, "attn_bwd: NULL pointer");
  if (((uintptr_t)scratch) & 15) return fail(TM_EALIGN, "attn_bwd: scratch must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  float *dvec = (float *)scratch;
  float *part = dvec + (batch * nq * seq + 63) / 64 * 64;
  if (int e = attn_dvec_launch(dtype, seq, batch, nq, nkv, d, ctx, dctx, dvec, s)) return e;
  if (rows_pay(dtype, true, seq, batch * nq, d) || !tiles_take(dtype, d, qkv, dqkv) || !tiles_take(dtype, d, dctx, dctx))
    return attn_bwd_generic_launch(dtype, seq, batch, nq, nkv, d, qkv, dctx, lse, dvec, dqkv, s);
  if (attn_mfma_supported(dtype, seq, batch, nq, nkv, d))
    return attn_bwd_mfma_launch(seq, batch, nq, nkv, d, qkv, dctx, lse, dvec, part, dqkv, s);
  if (attn_f32_supported(dtype, seq, batch, nq, nkv, d))
    return attn_bwd_f32_launch(seq, batch, nq, nkv, d, qkv, dctx, lse, dvec, part, dqkv, s);
  return attn_bwd_generic_launch(dtype, seq, batch, nq, nkv, d, qkv, dctx, lse, dvec, dqkv, s);
}
