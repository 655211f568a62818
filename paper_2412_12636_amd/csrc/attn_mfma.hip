// Flash-style causal attention on the CDNA4 matrix cores (bf16 in, fp32 accumulate), head sizes up to 128.
//
// The s x s score matrix is never stored: a block walks tiles of 64 rows, keeps running row maxima
// and sums in registers (online softmax) and accumulates its outputs in MFMA accumulators.
//
// Transposed products.  Everything is formed transposed (S^T = K Q^T, O^T = V^T P^T, ...), so that
// in every 32x32 accumulator tile the lane index is the row that owns the softmax statistics (a query
// row in the forward and dQ kernels, a key row in the dK/dV kernel) and the 16 accumulator registers
// run along the reduction axis of the NEXT product.  A lane's 8 consecutive accumulator registers are
// then exactly the 8 reduction-axis values the next MFMA expects from it, under a fixed permutation of
// that axis (slot (half h, e) <-> offset 8*(e/4) + 4*h + e%4).  Row statistics need one cross-half
// exchange per tile and no row-wise shuffles.
//
// One tile format.  Every staged tile is [64 rows][128 or 64] bf16, row-major as in global memory, fetched
// straight into LDS (buffer_load ... lds), double buffered.  An operand that is needed with the tile's
// rows as MFMA rows is read with plain 16-byte LDS reads; an operand that is needed TRANSPOSED (V in
// O^T = V^T P^T, K in dQ^T = K^T dS^T, Q and dO in the dK/dV kernel) is read from the same tile with
// the transposing LDS read ds_read_b64_tr_b16, which can also deliver the permuted reduction order
// directly.  The chunk placement inside a row is chosen so that both kinds of read are free of bank
// conflicts.
//
// Gradients are accumulated without atomics: dQ by a block that owns 128 query rows; dK/dV by a block
// that owns 128 key rows and loops over all later query tiles of ONE query head.  With grouped-query
// attention (several query heads per kv head) each head's block writes an fp32 partial and a small
// kernel adds the partials of a group in head order (a block looping over the whole group instead would
// leave a chip of 256 compute units with seq/128 * kv heads blocks: 32 for a 4096-token sequence and one
// kv head).
#include <math.h>
#include <stdlib.h>

#include "attn.h"
#include "attn_rows.h"

namespace tmk {

typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int TILE = 64;             // rows of a staged tile
constexpr float kLog2e = 1.4426950408889634f;

// Head sizes.  DP: the head size rounded up to a multiple of 32, the width the products run at (32, 64, 96 or 128).
// EX = false: head size 128, probabilities and dS go to the second product as bf16.  EX = true: every other head size
// up to 128; columns from the head size to DP are staged as zeros, and probabilities and dS keep 16 significand bits
// (a bf16 value plus the bf16 of what it leaves, two MFMAs), fewer than the 24 of the kernels with one row per wave that
// these sizes ran on before.  The results do not show the difference: against 64 bits both are off by their rounding to bf16
// and by ctx's rounding in the row statistics D, 1.6e-3 forward and 1.7e-3 backward, and with keys or values offset by up to 64
// times their spread, where the gradients cancel, by the same 0.8 % to 17 % to four digits.  (A third term, all 24 bits: the
// same errors again, forward 30 -> 36 us, backward 74 -> 85 at the size below.)  Rows with a non-finite value: attn_rows.h.
// One wave per row out of L2 took 43.6 ms for a forward and backward pass over 2 sequences of 1500, 16 query and 4 kv heads
// of 64, where this form takes 0.10 ms (31 us forward, 70 backward).  Of the cycles in which a unit has waves the matrix
// cores are busy for 28 % (forward) and 46 % (backward), its three waves a SIMD issue vector instructions for 60 % and
// 68 %: bound by the vector ALU work of a tile step and the chain through it (S product, softmax, PV product, barrier).
//
// A staged tile: [64][128] bf16 for DP 96 and 128, [64][64] for DP 32 and 64 (half the LDS: three blocks a unit).
template <int DP> struct TileFmt {
  static constexpr int ROWB = DP > 64 ? 256 : 128;  // bytes per tile row
  static constexpr int CPR = ROWB / 16;             // 16-byte chunks per row
  static constexpr int BYTES = TILE * ROWB;
  // Position of chunk c in tile row `row` is c ^ key(row) (256-byte rows: chunk bit 1 is also folded into bit 3, so
  // that the two 16-lane groups of a half-wave use different 128-byte halves).  The key takes as many distinct values
  // over 16 consecutive rows as there are chunk positions (plain reads of one chunk column by 16 lanes hit 16 different
  // bank groups), and the 4 rows of a transposing read land in different windows: 32-byte windows of a 256-byte row
  // (key bits 2:1 = the row's low bits), 64-byte halves of 128-byte rows (key bit 2 = row bit 1; row bit 0 already
  // picks the half of the 256 bytes of banks).
  static __device__ __forceinline__ int key(int row) {
    if constexpr (DP > 64) return ((row & 3) << 1) | ((row >> 2) & 1) | (((row >> 3) & 1) << 3);
    else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
  }
  static __device__ __forceinline__ int unplace(int pc, int row) {
    const int t = pc ^ key(row);
    if constexpr (DP > 64) return t ^ (((t >> 1) & 1) << 3);
    else return t;
  }
};

struct FlashParams {
  const bf16 *qkv;
  const bf16 *dctx;
  bf16 *ctx;
  bf16 *dqkv;
  float *lse;
  const float *lse_in;
  const float *dvec;
  float *part;                   // grouped-query dK/dV partials [batch][nq][seq][2][d] fp32, or NULL
  int seq, batch, nq, nkv, row;  // row = (nq + 2 nkv) * d
  int d;                         // head size
  float scale;                   // 1 / sqrt(d)
  uint32_t qkv_bytes, ctx_bytes;
};

// ---- global -> LDS: one tile, 16 (DP > 64) or 8 wave-wide loads a block ------------------------------
template <int DP, bool EX, int NW, int KT = TILE> struct TileLoaderN {  // KT: rows of the tile
  using F = TileFmt<DP>;
  static constexpr int NL = KT * F::ROWB / 1024 / NW;  // wave-wide loads per wave and tile
  uint32_t voff[NL];
  // row_stride: elements between consecutive tile rows in global memory; d: head size
  __device__ __forceinline__ void init(int64_t row_stride, int d, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = (i * NW + wave) * 64 + lane;  // chunk position in the LDS tile
      const int row = idx / F::CPR, c = F::unplace(idx % F::CPR, row);
      // Columns past the head size, and rows so far behind the tile's first that no tensor (below 2 GiB) holds both: an
      // offset that stays outside whatever tile start is added.  (Cut off at 32 bits instead, such a row's offset would come
      // round to the tensor's front: one position of 50000 batch entries of 16 heads of 64 is 307 MB, 64 rows are 19 GB.)
      const int64_t off = ((int64_t)row * row_stride + c * 8) * 2;
      voff[i] = off >= 0x80000000LL || (EX && c * 8 >= d) ? 0x80000000u : (uint32_t)off;
    }
  }
  // rows0: element offset of tile row 0 (a multiple of the row stride, inside the tensor), base: element offset of column 0
  // inside a row (below the row stride).  The row part travels in the per-lane offset, which the
  // hardware checks against the buffer size, so rows past the tensor read as zero.  The sum stays below 2^32.
  __device__ __forceinline__ void issue(rsrc_t rs, char *tile, int64_t rows0, int64_t base, int wave) const {
    const uint32_t roff = (uint32_t)(rows0 * 2), soff = (uint32_t)(base * 2);
#pragma unroll
    for (int i = 0; i < NL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(tile + (i * NW + wave) * 1024), 16, voff[i] + roff, soff, 0,
                                               0);
  }
};

// Fragment reads.  Every lane-dependent part of an address fits one per-lane base (relative to the tile, which must
// start on a 256-byte boundary); what changes with the reduction slice, the 32-column block and the row group is an XOR
// of the 16-byte chunk index with a compile-time constant plus a multiple of the row pitch, so that one register per
// kind of read serves all of them (written through the placement function the compiler keeps one address register per
// read, about forty of them).
//
// A-operand fragment, tile rows as MFMA rows: row r32 + lane%32, reduction slots 16ks + 8hh + 0..7
template <int DP> __device__ __forceinline__ uint32_t rows_base(int lane) {
  const int l32 = lane & 31, hh = lane >> 5;
  return (uint32_t)(l32 * TileFmt<DP>::ROWB + ((hh ^ TileFmt<DP>::key(l32)) << 4));
}
template <int DP> __device__ __forceinline__ bf16x8 frag_rows_at(const char *tile, uint32_t base, int r32, int ks) {
  const uint32_t x = (uint32_t)(((2 * ks) ^ (DP > 64 ? (ks & 1) << 3 : 0)) << 4);  // chunk 2ks + hh sits at hh ^ key ^ this
  return *reinterpret_cast<const bf16x8 *>(tile + ((base ^ x) + (uint32_t)(r32 * TileFmt<DP>::ROWB)));
}
// A-operand fragment of the TRANSPOSED tile: MFMA row = tile column c32 + lane%32, reduction axis =
// tile rows 16kk .. 16kk+15 in the permuted order (slot (hh, e) <-> row 16kk + 8*(e/4) + 4hh + e%4).
// ds_read_b64_tr_b16: within 16 lanes, lane i receives element i%4 of the 8-byte pieces addressed by
// lanes i/4, i/4+4, i/4+8, i/4+12; lane s addresses tile[row0 + s/4][col0 + 4*(s%4) ..+3].
template <int DP> __device__ __forceinline__ uint32_t cols_base(int lane) {  // the lane's column piece and row inside a group of 8
  const int g = lane >> 4, s = lane & 15;
  const int col = 16 * (g & 1) + 4 * (s & 3), c = col >> 3, half = (col >> 2) & 1;
  const int r = 4 * (g >> 1) + (s >> 2);
  const int pl = c ^ TileFmt<DP>::key(r) ^ (DP > 64 ? ((c >> 1) & 1) << 3 : 0);
  return (uint32_t)(r * TileFmt<DP>::ROWB + (pl << 4) + (half << 3));
}
template <int DP> __device__ __forceinline__ bf16x8 frag_cols_at(const char *tile, uint32_t base, int c32, int kk) {
  union { s16x4 h[2]; bf16x8 v; } x;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    // chunk index: + 4 per 32 columns; row 8t + r: bit 3 of the key of a 256-byte row is t, bit 1 of a 128-byte row's
    const uint32_t xr = (uint32_t)(((c32 >> 3) ^ (t << (DP > 64 ? 3 : 1))) << 4);
    const char *a = tile + ((base ^ xr) + (uint32_t)((16 * kk + 8 * t) * TileFmt<DP>::ROWB));
    x.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a));
  }
  return x.v;
}
// B-operand fragments straight from global memory: 8 consecutive elements of row (lane%32) per step
template <int DP, bool EX>
__device__ __forceinline__ void load_row_frags(const bf16 *rowptr, bool valid, int d, int hh, bf16x8 (&f)[DP / 16]) {
#pragma unroll
  for (int ks = 0; ks < DP / 16; ++ks) {
    union { u32x4 u; bf16x8 v; } x;
    x.u = u32x4{0u, 0u, 0u, 0u};
    if (valid && (!EX || ks * 16 + hh * 8 < d)) x.u = *reinterpret_cast<const u32x4 *>(rowptr + ks * 16 + hh * 8);
    f[ks] = x.v;
  }
}
// 8 accumulator registers (v0..v0+7) -> bf16 B-operand fragment
__device__ __forceinline__ bf16x8 pack8(const f32x16 &a, int v0) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16)a[v0 + e];
  return r;
}
// what pack8 left behind: the next 8 significand bits.  The values are taken back out of the packed words: element by
// element the compiler converts each one a second time (235 -> 202 vector instructions for the exponentials and second
// product of a 64-key tile).
__device__ __forceinline__ bf16x8 pack8_rest(const f32x16 &a, const bf16x8 &hi, int v0) {
  bf16x8 r;
  const u32x4 w = __builtin_bit_cast(u32x4, hi);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    r[2 * e] = (bf16)(a[v0 + 2 * e] - __builtin_bit_cast(float, w[e] << 16));
    r[2 * e + 1] = (bf16)(a[v0 + 2 * e + 1] - __builtin_bit_cast(float, w[e] & 0xffff0000u));
  }
  return r;
}
// the larger of the two halves' values of a row (lanes l and l + 32), without a trip through LDS
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
// offset along the accumulator-row axis of register v in a 32x32 tile
__device__ __forceinline__ int acc_row(int v, int hh) { return 8 * (v >> 2) + 4 * hh + (v & 3); }

// writes O^T-style accumulators (rows = head-dim slots, lane = token row) to out[token][col0 + d]
template <int DP, bool EX>
__device__ __forceinline__ void store_transposed(const f32x16 (&acc)[DP / 32], float mul, bf16 *dst_row, int d, int hh) {
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      if (EX && dt * 32 + 8 * q4 >= d) continue;  // d is a multiple of 8
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16)(acc[dt][q4 * 4 + e] * mul);
      *reinterpret_cast<bf16x4 *>(dst_row + dt * 32 + 8 * q4 + 4 * hh) = o;
    }
}
// the same accumulators as fp32: part_row points at [d] floats of this lane's token
template <int DP, bool EX>
__device__ __forceinline__ void store_transposed_f32(const f32x16 (&acc)[DP / 32], float mul, float *part_row, int d, int hh) {
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      if (EX && dt * 32 + 8 * q4 >= d) continue;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = acc[dt][q4 * 4 + e] * mul;
      *reinterpret_cast<f32x4 *>(part_row + dt * 32 + 8 * q4 + 4 * hh) = o;
    }
}
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// =================================================================================================
// forward
// =================================================================================================
// One wave's work on one staged K / V tile of 64 keys for its 32 query rows (lane%32 = query row): S^T = K Q^T,
// online softmax, O^T += V^T P^T.  Only the last one or two tiles of a walk can hold a key index above a query
// index of the wave: only those pay for the mask.
// EX: exponents are taken relative to a whole number m, and m moves only when some row's maximum has risen more than kLead
// above it (probabilities stay below 2^(kLead + 1)): with m the running maximum itself a wave rescales its accumulators
// and row sums on nearly every tile of a walk of a few dozen (one of 32 rows sees a new maximum).  Powers of two: every
// rescaling is exact, and the row sum's exponent joins m at the end (fwd_finish), so that the logarithm that is left is of
// a number from 1/2 to 1.  2 x 1500 positions, 16 / 4 heads of 64: 32.2 -> 28.1 us.
// Head size 128 keeps the maximum, and rescales when some row saw it rise (by exactly 1 where not): a row's largest
// probability is then 1, which bf16 holds exactly; taken to a whole number ctx is 16 % further from 64 bits (2.29e-3, 1.98e-3).
constexpr float kLead = 8.f;
template <int DP> struct FwdRow {
  f32x16 o[DP / 32];
  float m, l;  // reference exponent, row sum (of this half of the wave)
};
template <int DP, bool EX, int KT = TILE>
__device__ __forceinline__ void fwd_tile(const char *kt, const char *vt, const bf16x8 (&qf)[DP / 16], FwdRow<DP> &r, int j0,
                                         int q0w, int q, int hh, float sc2, uint32_t rb, uint32_t cb) {
  f32x16 s[KT / 32];
#pragma unroll
  for (int t = 0; t < KT / 32; ++t) {
#pragma unroll
    for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < DP / 16; ++ks)
      s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_at<DP>(kt, rb, t * 32, ks), qf[ks], s[t], 0, 0, 0);
  }
  if (j0 + KT - 1 > q0w) {  // wave-uniform
#pragma unroll
    for (int t = 0; t < KT / 32; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + t * 32 + acc_row(v, hh) > q) s[t][v] = -INFINITY;
  }
  float mraw = -INFINITY;
#pragma unroll
  for (int t = 0; t < KT / 32; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) mraw = fmaxf(mraw, s[t][v]);
  const float mx = max_halves(mraw) * sc2;
  if (__builtin_amdgcn_ballot_w64(mx > (EX ? r.m + kLead : r.m)) != 0) {  // wave-uniform; the first tile: m is -inf
    const float m = fmaxf(r.m, EX ? __builtin_ceilf(mx) : mx), alpha = __builtin_amdgcn_exp2f(r.m - m);
    r.m = m;
    r.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) r.o[dt][v] *= alpha;
  }
  float ps = 0.f;
#pragma unroll
  for (int t = 0; t < KT / 32; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][v], sc2, -r.m));
      s[t][v] = e;
      ps += e;
    }
  r.l += ps;
#pragma unroll
  for (int kk = 0; kk < KT / 16; ++kk) {
    const bf16x8 pf = pack8(s[kk >> 1], 8 * (kk & 1));
    bf16x8 pr;
    if (EX) pr = pack8_rest(s[kk >> 1], pf, 8 * (kk & 1));
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt) {
      const bf16x8 vf = frag_cols_at<DP>(vt, cb, dt * 32, kk);
      r.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, r.o[dt], 0, 0, 0);
      if (EX) r.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pr, r.o[dt], 0, 0, 0);
    }
  }
}
template <int DP, bool EX>
__device__ __forceinline__ void fwd_finish(const FlashParams &p, FwdRow<DP> &r, int q, int n, int g, int lane) {
  const int hd = EX ? p.d : DP, hh = lane >> 5;
  r.l += __shfl_xor(r.l, 32, 64);
  const uint32_t redo = EX ? nonfinite_rows(nonfinite_trace(r.o, r.l * 0.f), q < p.seq) : 0u;  // see attn_rows.h
  if (q < p.seq && !((redo >> (q & 31)) & 1)) {
    const int64_t trow = (int64_t)q * p.batch + n;
    store_transposed<DP, EX>(r.o, 1.f / r.l, p.ctx + trow * (p.nq * hd) + g * hd, hd, hh);
    if (hh == 0)
      p.lse[((int64_t)n * p.nq + g) * p.seq + q] =
          EX ? row_lse(r.m + (float)__builtin_amdgcn_frexp_expf(r.l), __builtin_amdgcn_frexp_mantf(r.l)) : (r.m + log2f(r.l)) * 0.6931471805599453f;
  }
  if constexpr (EX)
    for (uint32_t m = redo; m; m &= m - 1) attn_row_fwd<bf16>(p, q - (lane & 31) + __builtin_ctz(m), g, n, lane);
}

// block = 32 NW query rows of one (batch entry, query head); wave = 32 query rows.  Four waves, two blocks per
// compute unit; or eight waves, one block: the same waves per unit, but every staged K / V tile serves twice the query
// rows, which halves the bytes a unit pulls from L2 into LDS per MFMA (what bounds the walk of a long sequence).
template <int DP, bool EX, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? (DP > 64 ? 2 : 4) : 1) void flash_fwd_kernel(const FlashParams p) {
  __shared__ __align__(1024) char lds[2][2][TileFmt<DP>::BYTES];  // [stage][K, V]
  constexpr int QB = 32 * NW;
  const int qt = gridDim.z - 1 - blockIdx.z, g = blockIdx.x, n = blockIdx.y;  // heads fastest, longest walks first
  const int kap = g / (p.nq / p.nkv), hd = EX ? p.d : DP;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int q0w = qt * QB + wave * 32;
  const int q = q0w + l32;
  const int64_t tstride = (int64_t)p.batch * p.row;  // elements between consecutive positions
  const int koff = p.nq * hd + kap * hd, voff = (p.nq + p.nkv) * hd + kap * hd;
  const rsrc_t rs = make_rsrc(p.qkv, p.qkv_bytes);
  TileLoaderN<DP, EX, NW> ld;
  ld.init(tstride, hd, wave, lane);

  bf16x8 qf[DP / 16];
  load_row_frags<DP, EX>(p.qkv + (int64_t)n * p.row + (int64_t)q * tstride + g * hd, q < p.seq, hd, hh, qf);

  FwdRow<DP> r;
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) r.o[dt][v] = 0.f;
  r.m = -INFINITY;
  r.l = 0.f;
  const float sc2 = p.scale * kLog2e;
  const uint32_t rb = rows_base<DP>(lane), cb = cols_base<DP>(lane);

  const int kv_end = (qt * QB + QB < p.seq) ? qt * QB + QB : p.seq;
  const int ntile = (kv_end + TILE - 1) / TILE;
  ld.issue(rs, lds[0][0], 0, (int64_t)n * p.row + koff, wave);
  ld.issue(rs, lds[0][1], 0, (int64_t)n * p.row + voff, wave);
  for (int jt = 0; jt < ntile; ++jt) {
    const int j0 = jt * TILE, cur = jt & 1;
    wait_loads();
    __builtin_amdgcn_s_barrier();  // tile jt is in LDS; everyone is done with the other stage
    if (jt + 1 < ntile) {
      const int64_t r0 = (int64_t)(j0 + TILE) * tstride;
      ld.issue(rs, lds[cur ^ 1][0], r0, (int64_t)n * p.row + koff, wave);
      ld.issue(rs, lds[cur ^ 1][1], r0, (int64_t)n * p.row + voff, wave);
    }
    if (j0 > q0w + 31) continue;  // every key of this tile lies after every query row of the wave
    fwd_tile<DP, EX>(lds[cur][0], lds[cur][1], qf, r, j0, q0w, q, hh, sc2, rb, cb);
  }
  wait_loads();
  fwd_finish<DP, EX>(p, r, q, n, g, lane);
}

// The same for grids of at most one block per compute unit (short sequences, few heads), where the chain of tile
// steps of the last query rows bounds the kernel: eight waves; waves w and w + 4 share a SIMD and 32 query rows
// and take the even and the odd key tiles, each with its own maximum, row sum and accumulators; at the end the odd
// side's state goes through LDS and the even side merges it (o = o1 2^(m1-m) + o2 2^(m2-m), the row sum alike).
// Half as many steps, and the two waves of a SIMD overlap each other's softmax and MFMA phases.
// NPAR = 4: blocks of 64 query rows, each group of 32 walked by four waves that take every fourth tile (of 32 keys for the
// wide head sizes, so that two stages of four tiles fit the LDS): a quarter of the steps, twice the blocks, for grids whose
// blocks of 128 leave units idle (2048 positions, 4 heads of 128: 38.7 -> 31.4 us; where the line lies: fwd_ways).
template <int DP, bool EX, int NPAR> struct SplitFmt {
  static constexpr int NG = 8 / NPAR, QB = 32 * NG, KT = NPAR == 4 && DP > 64 ? 32 : TILE;
  static constexpr int TB = KT * TileFmt<DP>::ROWB, STATE = ((DP / 32) * 16 + 2) * 64;  // floats of a wave's state
  static constexpr int TILES = 2 * NPAR * 2 * TB, LDS = TILES;
  static_assert(NG * (NPAR - 1) * STATE * 4 <= TILES, "the states fit where the tiles were");
};
template <int DP, bool EX, int NPAR>
__global__ __launch_bounds__(512, DP > 64 ? 1 : NPAR == 2 ? 4 : 2) void flash_fwd_split_kernel(const FlashParams p) {
  extern __shared__ __align__(1024) char smem[];  // [stage][parity][K, V] tiles
  using S = SplitFmt<DP, EX, NPAR>;
  constexpr int KT = S::KT, QB = S::QB, NG = S::NG;
  const int qt = gridDim.z - 1 - blockIdx.z, g = blockIdx.x, n = blockIdx.y;  // heads fastest, longest walks first
  const int kap = g / (p.nq / p.nkv), hd = EX ? p.d : DP;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qg = wave % NG, par = wave / NG;
  const int l32 = lane & 31, hh = lane >> 5;
  const int q0w = qt * QB + qg * 32;
  const int q = q0w + l32;
  const int64_t tstride = (int64_t)p.batch * p.row;
  const int koff = p.nq * hd + kap * hd, voff = (p.nq + p.nkv) * hd + kap * hd;
  const rsrc_t rs = make_rsrc(p.qkv, p.qkv_bytes);
  TileLoaderN<DP, EX, 8, KT> ld;
  ld.init(tstride, hd, wave, lane);
  auto tile = [&](int stage, int parity, int which) { return smem + ((stage * NPAR + parity) * 2 + which) * S::TB; };

  bf16x8 qf[DP / 16];
  load_row_frags<DP, EX>(p.qkv + (int64_t)n * p.row + (int64_t)q * tstride + g * hd, q < p.seq, hd, hh, qf);

  FwdRow<DP> r;
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) r.o[dt][v] = 0.f;
  r.m = -INFINITY;
  r.l = 0.f;
  const float sc2 = p.scale * kLog2e;
  const uint32_t rb = rows_base<DP>(lane), cb = cols_base<DP>(lane);

  const int kv_end = (qt * QB + QB < p.seq) ? qt * QB + QB : p.seq;
  const int ntile = (kv_end + KT - 1) / KT, nstep = (ntile + NPAR - 1) / NPAR;
  auto issue_step = [&](int step, int stage) {  // all parities' tiles; a tile past the walk's end is not fetched
#pragma unroll
    for (int parity = 0; parity < NPAR; ++parity) {
      const int jt = NPAR * step + parity;
      if (jt < ntile) {
        const int64_t r0 = (int64_t)jt * KT * tstride;
        ld.issue(rs, tile(stage, parity, 0), r0, (int64_t)n * p.row + koff, wave);
        ld.issue(rs, tile(stage, parity, 1), r0, (int64_t)n * p.row + voff, wave);
      }
    }
  };
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int cur = step & 1;
    wait_loads();
    __builtin_amdgcn_s_barrier();  // this step's tiles are in LDS; everyone is done with the other stage
    if (step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    const int jt = NPAR * step + par, j0 = jt * KT;
    if (jt >= ntile || j0 > q0w + 31) continue;
    fwd_tile<DP, EX, KT>(tile(cur, par, 0), tile(cur, par, 1), qf, r, j0, q0w, q, hh, sc2, rb, cb);
  }
  wait_loads();
  __syncthreads();  // the tiles are no longer needed: the other sides' states go where they were
  float *xch = reinterpret_cast<float *>(smem);  // [qg][parity - 1][o..., m, l][lane]
  if (par > 0) {
    float *x = xch + (size_t)(qg * (NPAR - 1) + par - 1) * S::STATE;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[(dt * 16 + v) * 64 + lane] = r.o[dt][v];
    x[(DP / 32) * 16 * 64 + lane] = r.m;
    x[((DP / 32) * 16 + 1) * 64 + lane] = r.l;
  }
  __syncthreads();
  if (par == 0) {
#pragma unroll
    for (int o = 0; o < NPAR - 1; ++o) {
      const float *x = xch + (size_t)(qg * (NPAR - 1) + o) * S::STATE;
      const float m2 = x[(DP / 32) * 16 * 64 + lane], l2 = x[((DP / 32) * 16 + 1) * 64 + lane];
      const float mm = fmaxf(r.m, m2);  // r.m is finite: this side always has key tile 0
      const float a1 = __builtin_amdgcn_exp2f(r.m - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
      r.m = mm;
      r.l = r.l * a1 + l2 * a2;
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) r.o[dt][v] = r.o[dt][v] * a1 + x[(dt * 16 + v) * 64 + lane] * a2;
    }
    fwd_finish<DP, EX>(p, r, q, n, g, lane);
  }
}

// =================================================================================================
// dQ: same walk as the forward pass; dQ^T += K^T dS^T
// =================================================================================================
// one wave, one staged K / V tile: probabilities from the stored log-sum-exp, dS = P (dP - D), dQ^T += K^T dS^T
// FROM_D: dP starts from -D, which saves the subtraction behind the product; where head size 128 runs two four-wave blocks a
// unit the registers that hold it cost more (8192 positions, 8 heads: the backward pass 507 -> 520 us).
template <int DP, bool EX, bool FROM_D>
__device__ __forceinline__ void dq_tile(const char *kt, const char *vt, const bf16x8 (&qf)[DP / 16],
                                        const bf16x8 (&dof)[DP / 16], f32x16 (&acc)[DP / 32], float lse2, float dq_d, int j0,
                                        int q0w, int q, int hh, float sc2, uint32_t rb, uint32_t cb) {
  f32x16 ds[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    f32x16 s, dp;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f, dp[v] = FROM_D ? -dq_d : 0.f;
#pragma unroll
    for (int ks = 0; ks < DP / 16; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_at<DP>(kt, rb, t * 32, ks), qf[ks], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_at<DP>(vt, rb, t * 32, ks), dof[ks], dp, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
      ds[t][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], sc2, -lse2)) * (FROM_D ? dp[v] : dp[v] - dq_d);
  }
  if (j0 + TILE - 1 > q0w) {  // wave-uniform: only the last one or two tiles can hold a key above a query
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + t * 32 + acc_row(v, hh) > q) ds[t][v] = 0.f;
  }
#pragma unroll
  for (int kk = 0; kk < TILE / 16; ++kk) {
    const bf16x8 df = pack8(ds[kk >> 1], 8 * (kk & 1));
    bf16x8 dr;
    if (EX) dr = pack8_rest(ds[kk >> 1], df, 8 * (kk & 1));
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt) {
      const bf16x8 kf = frag_cols_at<DP>(kt, cb, dt * 32, kk);
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, df, acc[dt], 0, 0, 0);
      if (EX) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, dr, acc[dt], 0, 0, 0);
    }
  }
}

// block = 128 query rows (tile qt) of one (batch entry, query head), four waves; lds: [stage][K, V] tiles, 64 KB.
// In a block of eight waves the other four only keep the barrier count (one barrier per key tile).
// NPAR = 2: eight waves, waves w and w + 4 share query rows and take the even and the odd key tiles ([stage][parity]
// tiles, twice the LDS); their sums meet through LDS, first side + second side.
template <int DP, bool EX, int NW, int NPAR = 1>
__device__ __forceinline__ void dq_block(const FlashParams &p, char *lds_base, int qt, int g, int n) {
  auto tile = [&](int stage, int parity, int which) { return lds_base + ((stage * NPAR + parity) * 2 + which) * TileFmt<DP>::BYTES; };
  constexpr int QB = 32 * NW;  // query rows of the block (NW = 8: see the forward kernel)
  const int kap = g / (p.nq / p.nkv), hd = EX ? p.d : DP;
  const int lane = threadIdx.x & 63, wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = NPAR == 1 ? wave_id : wave_id % NW, par = NPAR == 1 ? 0 : wave_id / NW;
  if (NPAR == 1 && wave >= NW) {
    const int kv_end_x = (qt * QB + QB < p.seq) ? qt * QB + QB : p.seq;
    const int ntile_x = (kv_end_x + TILE - 1) / TILE;
    for (int jt = 0; jt < ntile_x; ++jt) __builtin_amdgcn_s_barrier();
    return;
  }
  const int l32 = lane & 31, hh = lane >> 5;
  const int q0w = qt * QB + wave * 32;
  const int q = q0w + l32;
  const bool qvalid = q < p.seq;
  const int64_t tstride = (int64_t)p.batch * p.row;
  const int koff = p.nq * hd + kap * hd, voff = (p.nq + p.nkv) * hd + kap * hd;
  const int64_t cstride = (int64_t)p.batch * p.nq * hd;
  const rsrc_t rs = make_rsrc(p.qkv, p.qkv_bytes);
  TileLoaderN<DP, EX, NW * NPAR> ld;
  ld.init(tstride, hd, wave_id, lane);

  bf16x8 qf[DP / 16], dof[DP / 16];
  load_row_frags<DP, EX>(p.qkv + (int64_t)n * p.row + (int64_t)q * tstride + g * hd, qvalid, hd, hh, qf);
  load_row_frags<DP, EX>(p.dctx + (int64_t)n * p.nq * hd + (int64_t)q * cstride + g * hd, qvalid, hd, hh, dof);
  const int64_t si = ((int64_t)n * p.nq + g) * p.seq + q;
  const float lse2 = qvalid ? p.lse_in[si] * kLog2e : 0.f;
  const float dq_d = qvalid ? p.dvec[si] : 0.f;

  f32x16 acc[DP / 32];
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[dt][v] = 0.f;
  const float sc2 = p.scale * kLog2e;
  const uint32_t rb = rows_base<DP>(lane), cb = cols_base<DP>(lane);

  const int kv_end = (qt * QB + QB < p.seq) ? qt * QB + QB : p.seq;
  const int ntile = (kv_end + TILE - 1) / TILE;
  auto issue_step = [&](int step, int stage) {
#pragma unroll
    for (int parity = 0; parity < NPAR; ++parity) {
      const int jt = NPAR * step + parity;
      if (NPAR == 1 || jt < ntile) {
        const int64_t r0 = (int64_t)jt * TILE * tstride;
        ld.issue(rs, tile(stage, parity, 0), r0, (int64_t)n * p.row + koff, wave_id);
        ld.issue(rs, tile(stage, parity, 1), r0, (int64_t)n * p.row + voff, wave_id);
      }
    }
  };
  const int nstep = (ntile + NPAR - 1) / NPAR;
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int jt = NPAR * step + par, j0 = jt * TILE, cur = step & 1;
    wait_loads();
    __builtin_amdgcn_s_barrier();
    if (step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    if ((NPAR > 1 && jt >= ntile) || j0 > q0w + 31) continue;
    dq_tile<DP, EX, EX || NPAR == 2 || NW == 8>(tile(cur, par, 0), tile(cur, par, 1), qf, dof, acc, lse2, dq_d, j0, q0w, q, hh, sc2, rb, cb);
  }
  wait_loads();
  if constexpr (NPAR == 2) {
    float *xch = reinterpret_cast<float *>(lds_base) + (size_t)wave * (DP / 32) * 16 * 64;  // [wave][dt][v][lane]
    __syncthreads();
    if (par == 1) {
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) xch[(dt * 16 + v) * 64 + lane] = acc[dt][v];
    }
    __syncthreads();
    if (par == 1) return;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[dt][v] += xch[(dt * 16 + v) * 64 + lane];
  }
  const uint32_t redo = EX ? nonfinite_rows(nonfinite_trace(acc, 0.f), qvalid) : 0u;  // see attn_rows.h
  if (qvalid && !((redo >> l32) & 1))
    store_transposed<DP, EX>(acc, p.scale, p.dqkv + ((int64_t)q * p.batch + n) * p.row + g * hd, hd, hh);
  if constexpr (EX)
    for (uint32_t m = redo; m; m &= m - 1) attn_row_dq<bf16>(p, q0w + __builtin_ctz(m), g, n, lane);
}
template <int DP, bool EX, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? (DP > 64 ? 2 : 3) : 1) void flash_bwd_dq_kernel(const FlashParams p) {
  __shared__ __align__(1024) char lds[4 * TileFmt<DP>::BYTES];
  const int qt = gridDim.z - 1 - blockIdx.z, g = blockIdx.x, n = blockIdx.y;  // heads fastest, longest walks first
  dq_block<DP, EX, NW>(p, lds, qt, g, n);
}

// =================================================================================================
// dK, dV: block = 128 key rows of one (batch entry, query head), eight waves: wave = 32 key rows x one 32-query
// half of every 64-row query tile (waves w and w + 4 share a SIMD and the key rows and take the two halves);
// loops over the query tiles from the diagonal to the end.  The two halves' sums over their queries are added
// through LDS at the end (first half + second half: a fixed order).  One query head per kv head: the block's
// result is the gradient.  Grouped heads: it is that head's fp32 partial.
// =================================================================================================
// smem: [stage][Q, dO] tiles, then [stage][lse, D] rows of floats, then the V fragments (kDkvLds bytes)
template <int DP, int NKR = 4, int NPAR = 1>
constexpr int kDkvLds = NPAR * (4 * TileFmt<DP>::BYTES + 2 * 2 * TILE * (int)sizeof(float)) + 32 * NKR * DP * 2;
// NKR: 32-key-row groups of the block, two waves each; NPAR = 2: four waves each, which share the walk as even and odd
// query tiles ([stage][parity] tiles and statistics, twice the LDS)
template <int DP, bool EX, int NKR = 4, int NPAR = 1>
__device__ __forceinline__ void dkv_block(const FlashParams &p, char *smem, int kt, int g, int n) {
  const int group = p.nq / p.nkv, kap = g / group, hd = EX ? p.d : DP;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kr = wave % NKR, t = NPAR == 1 ? wave / NKR : (wave / NKR) & 1;  // key-row group, query half
  const int par = NPAR == 1 ? 0 : wave / (2 * NKR);                          // even or odd query tiles
  const int l32 = lane & 31, hh = lane >> 5;
  const int j0w = kt * (32 * NKR) + kr * 32;
  const int j = j0w + l32;
  const bool jvalid = j < p.seq;
  const int64_t tstride = (int64_t)p.batch * p.row;
  const int koff = p.nq * hd + kap * hd, voff = (p.nq + p.nkv) * hd + kap * hd;
  const int64_t cstride = (int64_t)p.batch * p.nq * hd;
  const rsrc_t rq = make_rsrc(p.qkv, p.qkv_bytes), rdo = make_rsrc(p.dctx, p.ctx_bytes);
  TileLoaderN<DP, EX, 2 * NKR * NPAR> lq, ldo;
  lq.init(tstride, hd, wave, lane);
  ldo.init(cstride, hd, wave, lane);
  auto tile = [&](int stage, int parity, int which) { return smem + ((stage * NPAR + parity) * 2 + which) * TileFmt<DP>::BYTES; };
  float *stats = reinterpret_cast<float *>(smem + NPAR * 4 * TileFmt<DP>::BYTES);  // [stage][parity][2][TILE]

  // The wave's K fragments stay in registers; its V fragments live in LDS ([key-row group][slice][lane], 16 bytes
  // each: 32 KB a block, written once by the first query half) and are read again at every use, which keeps the
  // kernel inside 256 registers without spills.
  bf16x8 kf[DP / 16];
  load_row_frags<DP, EX>(p.qkv + (int64_t)n * p.row + (int64_t)j * tstride + koff, jvalid, hd, hh, kf);
  char *vl = smem + NPAR * (4 * TileFmt<DP>::BYTES + 2 * 2 * TILE * (int)sizeof(float)) + (kr * (DP / 16) * 64 + lane) * 16;
  if (t == 0 && par == 0) {
    bf16x8 vf[DP / 16];
    load_row_frags<DP, EX>(p.qkv + (int64_t)n * p.row + (int64_t)j * tstride + voff, jvalid, hd, hh, vf);
#pragma unroll
    for (int ks = 0; ks < DP / 16; ++ks) *reinterpret_cast<bf16x8 *>(vl + ks * 64 * 16) = vf[ks];
  }

  f32x16 dk[DP / 32], dv[DP / 32];
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) dk[dt][v] = dv[dt][v] = 0.f;
  const float sc2 = p.scale * kLog2e;
  const uint32_t rb = rows_base<DP>(lane), cb = cols_base<DP>(lane);

  const int it_begin = (kt * (32 * NKR)) / TILE;
  const int it_end = (p.seq + TILE - 1) / TILE;
  const int total = it_end - it_begin;
  // the query tiles of this head, double buffered; the row statistics of a step are fetched into registers one
  // step ahead by the first wave and put into LDS just before the barrier that publishes the step's tiles
  float st_lse = 0.f, st_d = 0.f;
  const int st_par = NPAR == 1 ? 0 : threadIdx.x / TILE, st_row = NPAR == 1 ? threadIdx.x : threadIdx.x % TILE;
  auto issue_step = [&](int step, int stage) {
#pragma unroll
    for (int parity = 0; parity < NPAR; ++parity) {
      const int it = NPAR * step + parity, i0 = (it_begin + it) * TILE;
      if (NPAR == 1 || it < total) {
        lq.issue(rq, tile(stage, parity, 0), (int64_t)i0 * tstride, (int64_t)n * p.row + g * hd, wave);
        ldo.issue(rdo, tile(stage, parity, 1), (int64_t)i0 * cstride, (int64_t)n * p.nq * hd + g * hd, wave);
      }
    }
    if (threadIdx.x < NPAR * TILE) {
      const int i = (it_begin + NPAR * step + st_par) * TILE + st_row;
      const int64_t sidx = ((int64_t)n * p.nq + g) * p.seq + i;
      st_lse = i < p.seq ? p.lse_in[sidx] * kLog2e : 0.f;
      st_d = i < p.seq ? p.dvec[sidx] : 0.f;
    }
  };
  const int nstep = (total + NPAR - 1) / NPAR;
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int cur = step & 1, it = NPAR * step + par;
    const int i0 = (it_begin + it) * TILE;
    wait_loads();
    if (threadIdx.x < NPAR * TILE) {
      float *st = stats + (cur * NPAR + st_par) * 2 * TILE;
      st[st_row] = st_lse;
      st[TILE + st_row] = st_d;
    }
    __syncthreads();  // tiles and statistics of this step are visible; the other stage is free
    if (step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    if (NPAR > 1 && it >= total) continue;
    if (i0 + t * 32 + 31 < j0w) continue;  // every query of this wave's half lies before every key row of the wave
    const char *qt = tile(cur, par, 0), *dot = tile(cur, par, 1);
    const float *lse_s = stats + (cur * NPAR + par) * 2 * TILE, *dv_s = lse_s + TILE;

    const bool diag = i0 + t * 32 < j0w + 31;  // some query index may be below some key index
    f32x16 s, dp;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = dp[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < DP / 16; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_at<DP>(qt, rb, t * 32, ks), kf[ks], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_at<DP>(dot, rb, t * 32, ks), *reinterpret_cast<const bf16x8 *>(vl + ks * 64 * 16), dp, 0, 0, 0);
    }
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int ib = t * 32 + 8 * q4 + 4 * hh;  // four consecutive query rows of this lane
      const f32x4 l4 = *reinterpret_cast<const f32x4 *>(lse_s + ib);
      const f32x4 d4 = *reinterpret_cast<const f32x4 *>(dv_s + ib);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = q4 * 4 + e;
        const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], sc2, -l4[e]));
        s[v] = x;                     // P
        dp[v] = x * (dp[v] - d4[e]);  // dS
      }
    }
    if (diag) {  // wave-uniform: only the first tiles of the walk can hold a query below a key of the wave
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (i0 + t * 32 + acc_row(v, hh) < j) s[v] = dp[v] = 0.f;
    }
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const int kk = 2 * t + k2;
      const bf16x8 pf = pack8(s, 8 * k2);
      const bf16x8 df = pack8(dp, 8 * k2);
      bf16x8 pr, dr;
      if (EX) pr = pack8_rest(s, pf, 8 * k2), dr = pack8_rest(dp, df, 8 * k2);
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt) {
        const bf16x8 dof = frag_cols_at<DP>(dot, cb, dt * 32, kk);
        dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dof, pf, dv[dt], 0, 0, 0);
        if (EX) dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dof, pr, dv[dt], 0, 0, 0);
        const bf16x8 qf = frag_cols_at<DP>(qt, cb, dt * 32, kk);
        dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, df, dk[dt], 0, 0, 0);
        if (EX) dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, dr, dk[dt], 0, 0, 0);
      }
    }
  }
  wait_loads();
  // (EX: from here on with the lane and what follows from it formed anew, which keeps them out of the loop's registers; for
  // head size 128 in bf16 the same costs four spilled ones, 4 % of its backward pass)
  const int tl = EX ? (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) : lane;
  const int tj = EX ? j0w + (tl & 31) : j;
  // the other query halves (and parities) hand their sums to the first through LDS (the tiles are no longer needed), dK,
  // then dV: added in the order first half, second half, the odd tiles' halves
  constexpr int NSIDE = 2 * NPAR;
  const int side = par * 2 + t;
  float *xch = reinterpret_cast<float *>(smem) + (size_t)kr * (NSIDE - 1) * (DP / 32) * 16 * 64;  // [kr][side - 1][dt][v][lane]
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    if (side > 0) {
      float *x = xch + (size_t)(side - 1) * (DP / 32) * 16 * 64;
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) x[(dt * 16 + v) * 64 + tl] = which == 0 ? dk[dt][v] : dv[dt][v];
    }
    __syncthreads();
    if (side == 0) {
#pragma unroll
      for (int o = 0; o < NSIDE - 1; ++o)
#pragma unroll
        for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float other = xch[((size_t)o * (DP / 32) * 16 + dt * 16 + v) * 64 + tl];
            if (which == 0) dk[dt][v] += other;
            else dv[dt][v] += other;
          }
    }
  }
  if (side > 0) return;
  const uint32_t redo = EX ? nonfinite_rows(nonfinite_trace(dk, nonfinite_trace(dv, 0.f)), tj < p.seq) : 0u;  // see attn_rows.h
  if (tj < p.seq && !((redo >> (tl & 31)) & 1)) {
    if (p.part) {
      float *out = p.part + (((int64_t)n * p.nq + g) * p.seq + tj) * (2 * hd);
      store_transposed_f32<DP, EX>(dk, p.scale, out, hd, tl >> 5);
      store_transposed_f32<DP, EX>(dv, 1.f, out + hd, hd, tl >> 5);
    } else {
      bf16 *out = p.dqkv + ((int64_t)tj * p.batch + n) * p.row;
      store_transposed<DP, EX>(dk, p.scale, out + koff, hd, tl >> 5);
      store_transposed<DP, EX>(dv, 1.f, out + voff, hd, tl >> 5);
    }
  }
  if constexpr (EX)
    for (uint32_t m = redo; m; m &= m - 1) attn_row_dkv<bf16>(p, j0w + __builtin_ctz(m), g, n, tl);
}

template <int DP, bool EX>
__global__ __launch_bounds__(512, 1) void flash_bwd_dkv_kernel(const FlashParams p) {
  extern __shared__ __align__(1024) char smem[];
  const int kt = blockIdx.z, g = blockIdx.x, n = blockIdx.y;  // heads fastest, longest walks first
  dkv_block<DP, EX>(p, smem, kt, g, n);
}

// Both backward kernels in one launch, for grids that leave compute units idle (at most one block of each kind per
// unit): the dK/dV block of key tile r and the dQ block of query tile last - r alternate in dispatch order, both
// kinds longest first, so that the chip works on the two independent halves of the backward pass at once instead of
// waiting twice for a longest walk (2048 tokens, 12 heads: 192 + 192 blocks on 256 units).  Blocks of eight waves;
// in a dQ block four of them only keep the barrier count.
template <int DP, bool EX>
__global__ __launch_bounds__(512, 1) void flash_bwd_both_kernel(const FlashParams p) {
  extern __shared__ __align__(1024) char smem[];
  const int rank = blockIdx.z >> 1, tiles = gridDim.z >> 1, g = blockIdx.x, n = blockIdx.y;
  if (blockIdx.z & 1) dq_block<DP, EX, 4>(p, smem, tiles - 1 - rank, g, n);
  else dkv_block<DP, EX>(p, smem, rank, g, n);
}

// The backward pass of head sizes up to 64 in one launch: blocks of four waves, a dK/dV block of 64 key rows or a dQ block
// of 128 query rows, three of them on a unit (168 registers, 41 KB), two dK/dV blocks to every dQ block in dispatch order
// and both kinds longest walk first.  (With the wide head sizes' blocks, eight waves of 169 registers and one block a
// unit, two launches took 39 + 49 us on 2 sequences of 1500 positions, 16 heads of 64; this one takes 65.)
template <int DP, bool EX>
__global__ __launch_bounds__(256, 3) void flash_bwd_narrow_kernel(const FlashParams p) {
  extern __shared__ __align__(1024) char smem[];
  const int rank = blockIdx.z / 3, kind = blockIdx.z % 3, tiles = gridDim.z / 3, g = blockIdx.x, n = blockIdx.y;
  if (kind == 2) {
    dq_block<DP, EX, 4>(p, smem, tiles - 1 - rank, g, n);
  } else if ((2 * rank + kind) * 64 < p.seq) {
    dkv_block<DP, EX, 2>(p, smem, 2 * rank + kind, g, n);
  }
}

// The backward pass for grids that leave units idle even as a single launch (the line: bwd_form): every walk is shared by two sets of waves that take
// alternate tiles (dK/dV blocks of 64 key rows, dQ blocks of 128 query rows, eight waves each, one block a unit), which
// halves the longest chain of tile steps: what bounds the single launch is the chain of key tile 0's walk, about 2 us a step
// for 1 us of MFMAs.  Dispatch order as above.  (2048 positions, 4 heads of 128: 68 -> 50 us.)
template <int DP, bool EX>
__global__ __launch_bounds__(512, 1) void flash_bwd_split_kernel(const FlashParams p) {
  extern __shared__ __align__(1024) char smem[];
  const int rank = blockIdx.z / 3, kind = blockIdx.z % 3, tiles = gridDim.z / 3, g = blockIdx.x, n = blockIdx.y;
  if (kind == 2) {
    dq_block<DP, EX, 4, 2>(p, smem, tiles - 1 - rank, g, n);
  } else if ((2 * rank + kind) * 64 < p.seq) {
    dkv_block<DP, EX, 2, 2>(p, smem, 2 * rank + kind, g, n);
  }
}

// Every kernel of a family by name, ahead of the host code that takes its address.
#define TM_FLASH_FAMILY(DP, EX)                                                \
  template __global__ void flash_fwd_kernel<DP, EX, 4>(const FlashParams);     \
  template __global__ void flash_fwd_split_kernel<DP, EX, 2>(const FlashParams);  \
  template __global__ void flash_fwd_split_kernel<DP, EX, 4>(const FlashParams);  \
  template __global__ void flash_bwd_split_kernel<DP, EX>(const FlashParams);  \
  template __global__ void flash_bwd_dq_kernel<DP, EX, 4>(const FlashParams);  \
  template __global__ void flash_bwd_dkv_kernel<DP, EX>(const FlashParams);    \
  template __global__ void flash_bwd_both_kernel<DP, EX>(const FlashParams);
TM_FLASH_FAMILY(128, false)
template __global__ void flash_fwd_kernel<128, false, 8>(const FlashParams);
template __global__ void flash_bwd_dq_kernel<128, false, 8>(const FlashParams);
#define TM_FLASH_NARROW(DP)                                                    \
  template __global__ void flash_fwd_kernel<DP, true, 4>(const FlashParams);     \
  template __global__ void flash_fwd_split_kernel<DP, true, 2>(const FlashParams);  \
  template __global__ void flash_fwd_split_kernel<DP, true, 4>(const FlashParams);  \
  template __global__ void flash_bwd_split_kernel<DP, true>(const FlashParams);  \
  template __global__ void flash_bwd_narrow_kernel<DP, true>(const FlashParams);
TM_FLASH_NARROW(32)
TM_FLASH_NARROW(64)
TM_FLASH_FAMILY(96, true)
TM_FLASH_FAMILY(128, true)

// dK, dV of a kv head = sum of its query heads' partials, added in head order; thread = 4 columns
__global__ __launch_bounds__(256) void flash_dkv_reduce_kernel(const FlashParams p) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // over [batch][nkv][seq][2 * d / 4]
  const int D = p.d;
  const int64_t total = (int64_t)p.batch * p.nkv * p.seq * (2 * D / 4);
  if (idx >= total) return;
  const int c4 = (int)(idx % (2 * D / 4));
  const int64_t r = idx / (2 * D / 4);
  const int j = (int)(r % p.seq);
  const int kap = (int)((r / p.seq) % p.nkv), n = (int)(r / ((int64_t)p.seq * p.nkv));
  const int group = p.nq / p.nkv;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int gg = 0; gg < group; ++gg) {
    const float *src = p.part + (((int64_t)n * p.nq + kap * group + gg) * p.seq + j) * (2 * D) + c4 * 4;
    const f32x4 v = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += v[e];
  }
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (bf16)sum[e];
  const int which = c4 / (D / 4), col = (c4 % (D / 4)) * 4;  // 0: dK, 1: dV
  bf16 *out = p.dqkv + ((int64_t)j * p.batch + n) * p.row + (p.nq + which * p.nkv + kap) * D + col;
  *reinterpret_cast<bf16x4 *>(out) = o;
}

// Every bf16 head size up to 128, as long as 32-bit offsets reach the tensors and the grid holds the sequence (head size
// 128 reports what it cannot take itself; the other head sizes have the plain-ALU kernels behind them).
bool attn_mfma_supported(int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  if (dtype != TM_DTYPE_BF16 || d > 128) return false;
  return d == 128 || seq * batch * (nq + 2 * nkv) * d * 2 < (1LL << 31);
}

static FlashParams make_params(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  FlashParams p = {};
  p.seq = (int)seq;
  p.batch = (int)batch;
  p.nq = (int)nq;
  p.nkv = (int)nkv;
  p.d = (int)d;
  p.row = (int)((nq + 2 * nkv) * d);
  p.scale = (float)(1.0 / sqrt((double)d));
  p.qkv_bytes = (uint32_t)(seq * batch * p.row * 2);
  p.ctx_bytes = (uint32_t)(seq * batch * nq * d * 2);
  return p;
}

static int unit_count() {
  static int units = 0;
  if (!units) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        units <= 0)
      units = 256;
  }
  return units;
}

// Sets of waves among which the forward kernel shares a walk: four, in blocks of 64 query rows, where every such block has
// a unit to itself, or, with walks of 1024 positions and more, half of the units a second one after the first; two, in
// blocks of 128, where the grid leaves compute units without a second block (at most one block per unit; two for head sizes
// up to 64, of which two blocks of eight waves fit a unit); else one.  A sequence of one block has nothing to share four
// ways.  Measured, one / two / four sets: 2048 positions, 8 heads of 128 (256 blocks) 46.8 / 39.3 / 32.4 us, 12 heads (384)
// 51.0 / 42.4 / 34.8, 4096 and 8 (512) 87.5 / 71.4 / 63.0; heads of 64: 1024 x 2 and 16 heads (512) 26.6 / 20.9 / 18.8, but
// 512 x 4 and 16 (512) 16.8 / 14.4 / 15.0, 1500 x 2 and 16 (768) 38.5 / 31.1 / 32.8.
// TM_ATTN_SPLIT=0 / 1 / 2 in the environment forces 1 / 2 / 4 (tuning and test aid).
static int fwd_ways(const FlashParams &p, dim3 grid, int blocks_per_unit) {
  if (const char *e = getenv("TM_ATTN_SPLIT")) return e[0] == '2' ? 4 : e[0] == '1' ? 2 : 1;
  const int64_t deep = (int64_t)p.nq * p.batch * ceil_div(p.seq, 64);
  if (p.seq > 128 && deep <= (p.seq >= 1024 ? 2 : 1) * (int64_t)unit_count()) return 4;
  return (int64_t)grid.x * grid.y * grid.z <= (int64_t)unit_count() * blocks_per_unit ? 2 : 1;
}

// Blocks of 256 query rows (eight waves) for the forward and dQ walks of grids that still give every compute unit two
// such blocks.  TM_ATTN_WIDE=0 / 1 forces the choice.
static bool use_wide(int64_t seq, int64_t batch, int64_t nq) {
  if (const char *e = getenv("TM_ATTN_WIDE")) return e[0] == '1';
  return ceil_div(seq, 256) * batch * nq >= 2 * (int64_t)unit_count();
}

// The backward pass as two launches (0), as one that holds both kinds of blocks where neither fills the chip by itself (1),
// or as one of shared walks (2) where even those blocks, three per 128 positions, have a unit each, or, with walks of 1024
// (2048) positions and more, up to 3/2 (15/8) blocks a unit.  Short walks of the narrow head sizes stay with their own kernel.
// Measured, form 1 / 2: 2048 positions, 4 heads of 128 (192 blocks) 68.0 / 50.2 us, 8 heads (384) 69.5 / 53.6, 10 (480)
// 72.2 / 66.2, 12 (576) 74.4 / 79.4; 1024 and 16 heads (384) 44.2 / 40.4, 20 (480) 47.2 / 47.9; 512 x 2 and 8 heads (192) 36.2 / 31.6, 16 heads (384) 32.2 / 34.0; heads of 64: 2048
// and 8 (384) 50.6 / 41.6, 384 x 2 and 8 (144) 18.0 / 17.5, 192 x 4 and 8 (192) 15.1 / 15.7.
// TM_ATTN_BWD_BOTH=0 / 1 / 2 forces the choice.
static int bwd_form(const FlashParams &p, dim3 grid) {
  if (const char *e = getenv("TM_ATTN_BWD_BOTH")) return e[0] == '2' ? 2 : e[0] == '1' ? 1 : 0;
  const int64_t blocks = (int64_t)grid.x * grid.y * grid.z, units = unit_count();
  if (p.seq > (p.d > 64 ? 128 : 320) && 3 * blocks <= (p.seq >= 2048 ? units * 15 / 8 : p.seq >= 1024 ? units * 3 / 2 : units)) return 2;
  return blocks <= units ? 1 : 0;
}

static bool reserve_lds(const void *kernel, int bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <int DP, bool EX> static int launch_fwd(const FlashParams &p, dim3 grid, hipStream_t s) {
  const int ways = fwd_ways(p, grid, DP > 64 ? 1 : 2);
  if (ways == 4) {
    using S = SplitFmt<DP, EX, 4>;
    static_assert(S::QB == 64, "blocks of 64 query rows");
    static bool attr_set = false;  // one flag per kernel family
    if (!attr_set && !reserve_lds(reinterpret_cast<const void *>(&flash_fwd_split_kernel<DP, EX, 4>), S::LDS))
      return fail(TM_ELAUNCH, "flash_fwd: cannot reserve LDS");
    attr_set = true;
    g_last_kernel = "flash_fwd_split_kernel";
    flash_fwd_split_kernel<DP, EX, 4><<<dim3(grid.x, grid.y, (unsigned)ceil_div(p.seq, 64)), 512, S::LDS, s>>>(p);
  } else if (ways == 2) {
    constexpr int lds = SplitFmt<DP, EX, 2>::LDS;
    static bool attr_set = false;
    if (!attr_set && !reserve_lds(reinterpret_cast<const void *>(&flash_fwd_split_kernel<DP, EX, 2>), lds))
      return fail(TM_ELAUNCH, "flash_fwd: cannot reserve LDS");
    attr_set = true;
    g_last_kernel = "flash_fwd_split_kernel";
    flash_fwd_split_kernel<DP, EX, 2><<<grid, 512, lds, s>>>(p);
  } else {
    g_last_kernel = "flash_fwd_kernel";
    bool wide = false;
    if constexpr (!EX) {
      wide = use_wide(p.seq, p.batch, p.nq);
      if (wide)
        flash_fwd_kernel<DP, EX, 8><<<dim3(grid.x, grid.y, (unsigned)ceil_div(p.seq, 256)), 512, 0, s>>>(p);
    }
    if (!wide) flash_fwd_kernel<DP, EX, 4><<<grid, 256, 0, s>>>(p);
  }
  return check_launch("flash_fwd");
}

int attn_fwd_mfma_launch(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d, const void *qkv, void *ctx,
                         float *lse, hipStream_t s) {
  if (seq * batch * (nq + 2 * nkv) * d * 2 >= (1LL << 31)) return fail(TM_ESIZE, "flash_fwd: qkv tensor above 2 GiB");
  FlashParams p = make_params(seq, batch, nq, nkv, d);
  p.qkv = (const bf16 *)qkv;
  p.ctx = (bf16 *)ctx;
  p.lse = lse;
  if (ceil_div(seq, 128) > 65535 || batch > 65535) return fail(TM_ESIZE, "flash_fwd: sequence or batch too long for the grid");
  // Block order = dispatch order: all heads of the longest walk (last query tile) first, then the next shorter one.
  // With the heads outermost instead, a long sequence's late heads start their longest walks when the chip is
  // already draining (16384 tokens, 8 heads, 512 block slots: 408 tile steps end to end against 258 balanced).
  dim3 grid((unsigned)nq, (unsigned)batch, (unsigned)ceil_div(seq, 128));
  if (d == 128) return launch_fwd<128, false>(p, grid, s);
  if (d <= 32) return launch_fwd<32, true>(p, grid, s);
  if (d <= 64) return launch_fwd<64, true>(p, grid, s);
  if (d <= 96) return launch_fwd<96, true>(p, grid, s);
  return launch_fwd<128, true>(p, grid, s);
}

static int reduce_heads(const FlashParams &p, hipStream_t s) {  // grouped heads: the heads' partials of dK and dV
  if (p.part) {
    const int64_t total = (int64_t)p.batch * p.nkv * p.seq * (2 * p.d / 4);
    flash_dkv_reduce_kernel<<<(unsigned)ceil_div(total, (int64_t)256), 256, 0, s>>>(p);
  }
  return check_launch("flash_bwd");
}

// the split form where it applies: launched (true) or not
template <int DP, bool EX> static bool launch_bwd_split(const FlashParams &p, dim3 gq, hipStream_t s, int *status) {
  constexpr int dkv = kDkvLds<DP, 2, 2>, dq = 8 * TileFmt<DP>::BYTES, lds = dkv > dq ? dkv : dq;
  static_assert(lds <= 160 * 1024 && lds >= 2 * 3 * (DP / 32) * 16 * 64 * 4, "fits, and the other sides' sums do");
  if (3 * (int64_t)gq.z > 65535 || bwd_form(p, gq) != 2) return false;
  static bool attr_set = false;
  if (!attr_set && !reserve_lds(reinterpret_cast<const void *>(&flash_bwd_split_kernel<DP, EX>), lds)) {
    *status = fail(TM_ELAUNCH, "flash_bwd: cannot reserve LDS");
    return true;
  }
  attr_set = true;
  g_last_kernel = "flash_bwd_split_kernel";
  flash_bwd_split_kernel<DP, EX><<<dim3(gq.x, gq.y, 3 * gq.z), 512, lds, s>>>(p);
  *status = reduce_heads(p, s);
  return true;
}

template <int DP> static int launch_bwd_narrow(const FlashParams &p, dim3 gq, hipStream_t s) {
  constexpr int lds = kDkvLds<DP, 2>;
  static_assert(lds >= 4 * TileFmt<DP>::BYTES && lds >= 2 * (DP / 32) * 16 * 64 * 4, "the dQ block's tiles and the second half's sums fit");
  static_assert(lds <= 64 * 1024, "no LDS attribute needed");
  if (3 * (int64_t)gq.z > 65535) return fail(TM_ESIZE, "flash_bwd: sequence too long for the grid");
  int status = TM_OK;
  if (launch_bwd_split<DP, true>(p, gq, s, &status)) return status;
  g_last_kernel = "flash_bwd_narrow_kernel";
  flash_bwd_narrow_kernel<DP, true><<<dim3(gq.x, gq.y, 3 * gq.z), 256, lds, s>>>(p);
  return reduce_heads(p, s);
}

template <int DP, bool EX> static int launch_bwd(const FlashParams &p, dim3 gq, hipStream_t s) {
  int status = TM_OK;
  if (launch_bwd_split<DP, EX>(p, gq, s, &status)) return status;
  constexpr int lds = kDkvLds<DP>;
  static_assert(lds >= 4 * TileFmt<DP>::BYTES, "the dQ block's tiles fit the dK/dV block's LDS");
  static_assert(lds >= 4 * (DP / 32) * 16 * 64 * 4, "the second query half's sums fit");
  static bool attr_set = false;
  if (!attr_set && (!reserve_lds(reinterpret_cast<const void *>(&flash_bwd_dkv_kernel<DP, EX>), lds) ||
                    !reserve_lds(reinterpret_cast<const void *>(&flash_bwd_both_kernel<DP, EX>), lds)))
    return fail(TM_ELAUNCH, "flash_bwd: cannot reserve LDS");
  attr_set = true;
  g_last_kernel = "flash_bwd_dq_kernel+flash_bwd_dkv_kernel";
  if (bwd_form(p, gq) != 0 && 2 * gq.z <= 65535) {
    g_last_kernel = "flash_bwd_both_kernel";
    flash_bwd_both_kernel<DP, EX><<<dim3(gq.x, gq.y, 2 * gq.z), 512, lds, s>>>(p);
  } else {
    bool wide = false;
    if constexpr (!EX) {
      wide = use_wide(p.seq, p.batch, p.nq);
      if (wide)
        flash_bwd_dq_kernel<DP, EX, 8><<<dim3(gq.x, gq.y, (unsigned)ceil_div(p.seq, 256)), 512, 0, s>>>(p);
    }
    if (!wide) flash_bwd_dq_kernel<DP, EX, 4><<<gq, 256, 0, s>>>(p);
    flash_bwd_dkv_kernel<DP, EX><<<gq, 512, lds, s>>>(p);
  }
  return reduce_heads(p, s);
}

int64_t attn_bwd_mfma_partial_floats(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  return nq == nkv ? 0 : batch * nq * seq * 2 * d;
}

int attn_bwd_mfma_launch(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d, const void *qkv,
                         const void *dctx, const float *lse, const float *dvec, float *part, void *dqkv,
                         hipStream_t s) {
  if (seq * batch * (nq + 2 * nkv) * d * 2 >= (1LL << 31)) return fail(TM_ESIZE, "flash_bwd: qkv tensor above 2 GiB");
  FlashParams p = make_params(seq, batch, nq, nkv, d);
  p.qkv = (const bf16 *)qkv;
  p.dctx = (const bf16 *)dctx;
  p.lse_in = lse;
  p.dvec = dvec;
  p.dqkv = (bf16 *)dqkv;
  p.part = nq == nkv ? nullptr : part;
  if (nq != nkv && !part) return fail(TM_EINVAL, "flash_bwd: grouped heads need the partial buffer");
  if (ceil_div(seq, 128) > 65535 || batch > 65535) return fail(TM_ESIZE, "flash_bwd: sequence or batch too long for the grid");
  dim3 gq((unsigned)nq, (unsigned)batch, (unsigned)ceil_div(seq, 128));  // heads fastest: see the forward launch
  if (d == 128) return launch_bwd<128, false>(p, gq, s);
  if (d <= 32) return launch_bwd_narrow<32>(p, gq, s);
  if (d <= 64) return launch_bwd_narrow<64>(p, gq, s);
  if (d <= 96) return launch_bwd<96, true>(p, gq, s);
  return launch_bwd<128, true>(p, gq, s);
}

}  // namespace tmk
