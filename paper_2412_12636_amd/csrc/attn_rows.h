// Rows of causal attention one at a time on the plain ALUs, reading only the positions that take part in the row.
//
// The tiled kernels multiply whole tiles: a position that the causal mask excludes has probability 0, and 0 times an
// infinite or NaN entry of that position is NaN.  So they look at what they are about to store (one multiply-add per
// accumulator register, at the end of a walk), and a wave that holds a row with a non-finite value forms that row again
// here, from the definition.  Rows that only shared a tile with such a position get their finite values; rows that the
// position belongs to get what the definition gives for it.  The same catches a row of which a whole tile of scores is
// -Inf (the running maximum of the tiled form has no value then) and operands whose high part leaves the range of bf16.
#pragma once
#include <math.h>

#include "common.h"

namespace tmk {

template <int N, typename Acc> __device__ __forceinline__ float nonfinite_trace(const Acc (&acc)[N], float t) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) t = __builtin_fmaf(acc[i][v], 0.f, t);
  return t;  // 0, or NaN if a value is infinite or NaN
}
// the rows of a 32-row wave tile (lane % 32) of which either half-wave holds a non-finite value; every lane of the wave calls
__device__ __forceinline__ uint32_t nonfinite_rows(float trace, bool valid) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(valid && !(trace == 0.f));
  return (uint32_t)m | (uint32_t)(m >> 32);
}

// log-sum-exp of a row from the maximum m in exponent units (base 2) and the sum l: m ln 2 + ln l with one rounding behind it
// (ln 2 as its fp32 value and what that leaves)
__device__ __forceinline__ float row_lse(float m, float l) {
  return __builtin_fmaf(m, 0.693147182464599609375f, __builtin_fmaf(m, -1.904654323148236017e-09f, logf(l)));
}

template <typename T> __device__ __forceinline__ float row_dot(const T *a, const T *b, int d) {
  float s = 0.f;
  for (int e = 0; e < d; ++e) s = fmaf(to_f32(a[e]), to_f32(b[e]), s);
  return s;
}

// P: the parameter block of a tiled kernel.  One wave; head sizes up to 128 (two columns a lane).
template <typename T, typename P> __device__ __forceinline__ void attn_row_fwd(const P &p, int i, int g, int n, int lane) {
  const int d = p.d, kap = g / (p.nq / p.nkv);
  const int64_t ts = (int64_t)p.batch * p.row;
  const T *base = p.qkv + (int64_t)n * p.row, *q = base + (int64_t)i * ts + g * d;
  const T *k = base + (int64_t)(p.nq + kap) * d, *v = k + (int64_t)p.nkv * d;
  float mx = -INFINITY, sum = 0.f, o0 = 0.f, o1 = 0.f;
  for (int j = lane; j <= i; j += 64) mx = fmaxf(mx, row_dot(q, k + (int64_t)j * ts, d) * p.scale);
  mx = wave_max(mx);
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane, count = i - j0 < 63 ? i - j0 + 1 : 64;
    const float pj = j <= i ? expf(row_dot(q, k + (int64_t)j * ts, d) * p.scale - mx) : 0.f;
    sum += pj;
    for (int t = 0; t < count; ++t) {
      const float w = __shfl(pj, t, 64);
      const T *vr = v + (int64_t)(j0 + t) * ts;
      if (lane < d) o0 = fmaf(w, to_f32(vr[lane]), o0);
      if (lane + 64 < d) o1 = fmaf(w, to_f32(vr[lane + 64]), o1);
    }
  }
  sum = wave_sum(sum);
  const float inv = 1.f / sum;
  T *out = p.ctx + ((int64_t)i * p.batch + n) * (p.nq * d) + g * d;
  if (lane < d) out[lane] = from_f32<T>(o0 * inv);
  if (lane + 64 < d) out[lane + 64] = from_f32<T>(o1 * inv);
  if (lane == 0) p.lse[((int64_t)n * p.nq + g) * p.seq + i] = mx + logf(sum);
}

template <typename T, typename P> __device__ __forceinline__ void attn_row_dq(const P &p, int i, int g, int n, int lane) {
  const int d = p.d, kap = g / (p.nq / p.nkv);
  const int64_t ts = (int64_t)p.batch * p.row, si = ((int64_t)n * p.nq + g) * p.seq + i;
  const T *base = p.qkv + (int64_t)n * p.row, *q = base + (int64_t)i * ts + g * d;
  const T *k = base + (int64_t)(p.nq + kap) * d, *v = k + (int64_t)p.nkv * d;
  const T *dc = p.dctx + ((int64_t)i * p.batch + n) * (p.nq * d) + g * d;
  const float l = p.lse_in[si], D = p.dvec[si];
  float o0 = 0.f, o1 = 0.f;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane, count = i - j0 < 63 ? i - j0 + 1 : 64;
    float ds = 0.f;
    if (j <= i) ds = expf(row_dot(q, k + (int64_t)j * ts, d) * p.scale - l) * (row_dot(dc, v + (int64_t)j * ts, d) - D);
    for (int t = 0; t < count; ++t) {
      const float w = __shfl(ds, t, 64);
      const T *kr = k + (int64_t)(j0 + t) * ts;
      if (lane < d) o0 = fmaf(w, to_f32(kr[lane]), o0);
      if (lane + 64 < d) o1 = fmaf(w, to_f32(kr[lane + 64]), o1);
    }
  }
  T *out = p.dqkv + ((int64_t)i * p.batch + n) * p.row + g * d;
  if (lane < d) out[lane] = from_f32<T>(o0 * p.scale);
  if (lane + 64 < d) out[lane + 64] = from_f32<T>(o1 * p.scale);
}

// the share of query head g in row j of dK and dV: into the head's fp32 partial where query heads share kv heads
template <typename T, typename P> __device__ __forceinline__ void attn_row_dkv(const P &p, int j, int g, int n, int lane) {
  const int d = p.d, kap = g / (p.nq / p.nkv);
  const int64_t ts = (int64_t)p.batch * p.row, cs = (int64_t)p.batch * p.nq * d, stats = ((int64_t)n * p.nq + g) * p.seq;
  const T *base = p.qkv + (int64_t)n * p.row, *q = base + g * d;
  const T *k = base + (int64_t)j * ts + (int64_t)(p.nq + kap) * d, *v = k + (int64_t)p.nkv * d;
  const T *dc = p.dctx + (int64_t)n * p.nq * d + g * d;
  float dk0 = 0.f, dk1 = 0.f, dv0 = 0.f, dv1 = 0.f;
  for (int i0 = j; i0 < p.seq; i0 += 64) {
    const int i = i0 + lane, count = p.seq - i0 < 64 ? p.seq - i0 : 64;
    float pi = 0.f, ds = 0.f;
    if (i < p.seq) {
      pi = expf(row_dot(q + (int64_t)i * ts, k, d) * p.scale - p.lse_in[stats + i]);
      ds = pi * (row_dot(dc + (int64_t)i * cs, v, d) - p.dvec[stats + i]);
    }
    for (int t = 0; t < count; ++t) {
      const float wp = __shfl(pi, t, 64), wd = __shfl(ds, t, 64);
      const T *dr = dc + (int64_t)(i0 + t) * cs, *qr = q + (int64_t)(i0 + t) * ts;
      if (lane < d) dv0 = fmaf(wp, to_f32(dr[lane]), dv0), dk0 = fmaf(wd, to_f32(qr[lane]), dk0);
      if (lane + 64 < d) dv1 = fmaf(wp, to_f32(dr[lane + 64]), dv1), dk1 = fmaf(wd, to_f32(qr[lane + 64]), dk1);
    }
  }
  if (p.part) {
    float *out = p.part + (stats + j) * (2 * d);
    if (lane < d) out[lane] = dk0 * p.scale, out[d + lane] = dv0;
    if (lane + 64 < d) out[lane + 64] = dk1 * p.scale, out[d + lane + 64] = dv1;
  } else {
    T *out = p.dqkv + ((int64_t)j * p.batch + n) * p.row + (int64_t)(p.nq + kap) * d, *outv = out + (int64_t)p.nkv * d;
    if (lane < d) out[lane] = from_f32<T>(dk0 * p.scale), outv[lane] = from_f32<T>(dv0);
    if (lane + 64 < d) out[lane + 64] = from_f32<T>(dk1 * p.scale), outv[lane + 64] = from_f32<T>(dv1);
  }
}

}  // namespace tmk
