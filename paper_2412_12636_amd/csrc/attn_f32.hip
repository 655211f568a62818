// Flash-style causal attention of the fp32 stage dtype on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32
// accumulation), head sizes up to 128.
//
// Transposed products as in the bf16 kernels (S^T = K Q^T, O^T = V^T P^T, ...): in every 32x32 accumulator tile the lane
// index is the row that owns the softmax statistics and the 16 registers run along the reduction axis of the next
// product.  That product takes two reduction slots per MFMA, one from each half of the wave, so an accumulator register
// IS the operand of one MFMA: register v holds rows 8(v/4) + v%4 (first half) and the row 4 further on (second half).
//
// A block is four waves: two groups of 32 rows that it owns, times two sides that take the even and the odd 32-row tiles
// of its walk and meet through LDS at the end in a fixed order; or one group times four sides.  (Short sequences and few
// heads leave most SIMDs without a wave, so the walk is split rather than the block made larger.)  A tile is [32 rows][DP]
// fp32, fetched straight into LDS by one wave (DP = head size rounded up to 32; columns and rows past the tensor read as
// zero), double buffered (the wide head sizes on four sides: one buffer).
//
// Bound by the MFMA rate, 64 clocks each, DP of them per tile and wave in the forward pass against about 150 vector
// instructions and LDS reads of one 16-byte or four 4-byte words per four MFMAs, and by how few waves a short sequence
// gives a SIMD: over 2 x 512 positions, 16 heads of 64, the matrix cores are busy for 64 % (backward) of the cycles in which
// a unit has waves and, with one wave a SIMD, 45 % (forward).  (One wave per row with every operand out of L2 took 5.4 ms
// for both passes, this form takes 0.095.)  Rows with a non-finite value: attn_rows.h.
#include <math.h>

#include "attn.h"
#include "attn_rows.h"

namespace tmk {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int FT = 32;   // rows of a staged tile
constexpr float kLog2ef = 1.4426950408889634f;

struct F32Params {
  const float *qkv, *dctx, *lse_in, *dvec;
  float *ctx, *dqkv, *lse;
  float *part;                      // grouped-query dK/dV partials [batch][nq][seq][2][d], or NULL
  int seq, batch, nq, nkv, d, row;  // row = (nq + 2 nkv) * d
  float scale;
  uint32_t qkv_bytes, ctx_bytes;
};

// 16-byte chunk c of tile row r sits at c ^ key(r): 16 rows read at one chunk column use 16 different bank groups.
template <int DP> struct F32Tile {
  static constexpr int ROWB = DP * 4, CPR = DP / 4, BYTES = FT * ROWB, NL = BYTES / 1024;
  static constexpr bool WIDE = CPR % 16 == 0;  // row pitch a multiple of 256 bytes
  static __device__ __forceinline__ int key(int r) { return WIDE ? r & 15 : (r >> 1) & 7; }
  // the part of key(8 (v/4) + 4 hh + v%4) that depends on the register only; the rest is 4 hh (WIDE) or 2 hh
  static constexpr __device__ __forceinline__ int key_v(int v) {
    return WIDE ? (8 * ((v >> 2) & 1)) | (v & 3) : (4 * ((v >> 2) & 1)) | ((v >> 1) & 1);
  }
};

// one wave fetches one tile
template <int DP> struct F32Loader {
  using F = F32Tile<DP>;
  uint32_t voff[F::NL];
  __device__ __forceinline__ void init(int64_t row_stride, int d, int lane) {
#pragma unroll
    for (int i = 0; i < F::NL; ++i) {
      const int idx = i * 64 + lane, r = idx / F::CPR, c = (idx % F::CPR) ^ F::key(r);
      // columns past the head size, and rows so far behind the tile's first that no tensor (below 2 GiB) holds both: an
      // offset that stays outside, and below 2^32, whatever tile start inside the tensor is added
      const int64_t off = (r * row_stride + c * 4) * 4;
      voff[i] = c * 4 < d && off < 0x80000000LL ? (uint32_t)off : 0x80000000u;
    }
  }
  __device__ __forceinline__ void issue(rsrc_t rs, char *tile, int64_t row0, int64_t base) const {
#pragma unroll
    for (int i = 0; i < F::NL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(tile + i * 1024), 16, voff[i] + (uint32_t)(row0 * 4),
                                               (uint32_t)(base * 4), 0, 0);
  }
};

// A operand, tile rows as MFMA rows: four reduction slots 8j + 4hh .. +3 of row lane%32
template <int DP> __device__ __forceinline__ f32x4 f32_rows(const char *tile, int j, int lane) {
  const int r = lane & 31, hh = lane >> 5;
  return *reinterpret_cast<const f32x4 *>(tile + r * F32Tile<DP>::ROWB + (((2 * j + hh) ^ F32Tile<DP>::key(r)) << 4));
}
// A operand of the transposed tile: MFMA row = column c32 + lane%32, reduction slot = row 8(v/4) + 4hh + v%4
template <int DP> __device__ __forceinline__ uint32_t f32_cols_base(int lane) {
  using F = F32Tile<DP>;
  const int l32 = lane & 31, hh = lane >> 5;
  return (uint32_t)((((l32 >> 2) ^ (F::WIDE ? 4 * hh : 2 * hh)) << 4) + ((l32 & 3) << 2) + hh * 4 * F::ROWB);
}
template <int DP> __device__ __forceinline__ float f32_cols(const char *tile, uint32_t base, int c32, int v) {
  using F = F32Tile<DP>;
  const uint32_t x = (uint32_t)(((c32 >> 2) ^ F::key_v(v)) << 4);
  return *reinterpret_cast<const float *>(tile + ((base ^ x) + (uint32_t)((8 * (v >> 2) + (v & 3)) * F::ROWB)));
}
// B operand from global memory: the lane's row, reduction slots 8j + 4hh .. +3
template <int DP> __device__ __forceinline__ void f32_row_frags(const float *row, bool valid, int d, int hh, f32x4 (&f)[DP / 8]) {
#pragma unroll
  for (int j = 0; j < DP / 8; ++j) {
    f[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (valid && 8 * j < d) f[j] = *reinterpret_cast<const f32x4 *>(row + 8 * j + 4 * hh);
  }
}
__device__ __forceinline__ f32x16 f32_zero() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
// acc (rows = tile rows, lane = own row) = tile . own rows
template <int DP> __device__ __forceinline__ f32x16 f32_scores(const char *tile, const f32x4 (&own)[DP / 8], int lane) {
  f32x16 s = f32_zero();
#pragma unroll
  for (int j = 0; j < DP / 8; ++j) {
    const f32x4 a = f32_rows<DP>(tile, j, lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], own[j][i], s, 0, 0, 0);
  }
  return s;
}
// acc[dt] (rows = columns of the tile, lane = own row) += tile^T . w
template <int DP> __device__ __forceinline__ void f32_accumulate(const char *tile, uint32_t cb, const f32x16 &w, f32x16 (&acc)[DP / 32]) {
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(f32_cols<DP>(tile, cb, dt * 32, v), w[v], acc[dt], 0, 0, 0);
}
__device__ __forceinline__ int f32_acc_row(int v, int hh) { return 8 * (v >> 2) + 4 * hh + (v & 3); }
template <int DP> __device__ __forceinline__ void f32_store(const f32x16 (&acc)[DP / 32], float mul, float *dst, int d, int hh) {
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      if (dt * 32 + 8 * q4 >= d) continue;  // d is a multiple of 8
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = acc[dt][q4 * 4 + e] * mul;
      *reinterpret_cast<f32x4 *>(dst + dt * 32 + 8 * q4 + 4 * hh) = o;
    }
}
__device__ __forceinline__ void f32_wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// How a block's four waves share its walk.  SIDES = 2: two groups of 32 rows, each with an even and an odd side; a wave
// fetches one of a step's four tiles.  SIDES = 4: one group, every wave takes each fourth tile and fetches its own, so the
// waves meet only at the end.
template <int DP, int SIDES> struct F32Walk {
  static constexpr int GROUPS = 4 / SIDES, FB = 32 * GROUPS;  // FB: rows a block owns
  static constexpr int NST = SIDES == 2 || DP <= 64 ? 2 : 1;  // LDS stages
  static constexpr int TILES = NST * SIDES * 2 * F32Tile<DP>::BYTES;
  static constexpr int LDS = TILES + NST * SIDES * 2 * FT * (int)sizeof(float);  // and the row statistics of dK / dV
  static_assert((SIDES - 1) * GROUPS * (DP / 2 + 2) * 256 <= TILES, "the sides' sums fit where the tiles were");
  // the next step's loads may be issued behind this: everyone who uses a tile of that stage is done with it
  static __device__ __forceinline__ void publish() {
    if constexpr (SIDES == 2) __syncthreads();
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
};
// the later sides' accumulators are added to the first's through LDS in order (x: this group's [side][DP / 32][16][64] floats)
template <int DP, int SIDES> __device__ __forceinline__ void f32_join(f32x16 (&acc)[DP / 32], float *x, int side, int lane) {
  __syncthreads();
  if (side > 0) {
    const int at = SIDES == 2 ? 0 : (side - 1) * (DP / 2);
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) x[(at + dt * 16 + v) * 64 + lane] = acc[dt][v];
  }
  __syncthreads();
  if (side == 0) {
#pragma unroll
    for (int o = 0; o < SIDES - 1; ++o)
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[dt][v] += x[(o * (DP / 2) + dt * 16 + v) * 64 + lane];
  }
}

// ---- forward: block = FB query rows of one (batch entry, query head) ----------------------------------
template <int DP, int SIDES> __global__ __launch_bounds__(256, 1) void f32_fwd_kernel(const F32Params p) {
  extern __shared__ __align__(1024) char smem[];  // [stage][side][K, V]
  using F = F32Tile<DP>;
  using W = F32Walk<DP, SIDES>;
  constexpr int FB = W::FB, NST = W::NST;
  const int qt = gridDim.z - 1 - blockIdx.z, g = blockIdx.x, n = blockIdx.y;  // heads fastest, longest walks first
  const int kap = g / (p.nq / p.nkv), d = p.d;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave % W::GROUPS, side = wave / W::GROUPS, l32 = lane & 31, hh = lane >> 5;
  const int q0w = qt * FB + grp * 32, q = q0w + l32;
  const int64_t ts = (int64_t)p.batch * p.row;
  const int koff = (p.nq + kap) * d, voff = (p.nq + p.nkv + kap) * d;
  const rsrc_t rs = make_rsrc(p.qkv, p.qkv_bytes);
  F32Loader<DP> ld;
  ld.init(ts, d, lane);
  auto tile = [&](int stage, int s, int which) { return smem + ((stage * SIDES + s) * 2 + which) * F::BYTES; };
  f32x4 qf[DP / 8];
  f32_row_frags<DP>(p.qkv + (int64_t)n * p.row + (int64_t)q * ts + g * d, q < p.seq, d, hh, qf);
  f32x16 o[DP / 32];
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt) o[dt] = f32_zero();
  float m = -INFINITY, l = 0.f;
  const float sc2 = p.scale * kLog2ef;
  const uint32_t cb = f32_cols_base<DP>(lane);
  const int kv_end = qt * FB + FB < p.seq ? qt * FB + FB : p.seq;
  const int ntile = (kv_end + FT - 1) / FT, nstep = (ntile + SIDES - 1) / SIDES;
  auto issue_step = [&](int step, int stage) {  // no tile past the walk's end
    if constexpr (SIDES == 2) {
      const int s = wave >> 1, which = wave & 1, jt = 2 * step + s;
      if (jt < ntile) ld.issue(rs, tile(stage, s, which), (int64_t)jt * FT * ts, (int64_t)n * p.row + (which ? voff : koff));
    } else {
      const int jt = SIDES * step + side;
      if (jt < ntile) {
        ld.issue(rs, tile(stage, side, 0), (int64_t)jt * FT * ts, (int64_t)n * p.row + koff);
        ld.issue(rs, tile(stage, side, 1), (int64_t)jt * FT * ts, (int64_t)n * p.row + voff);
      }
    }
  };
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int cur = NST == 2 ? step & 1 : 0, jt = SIDES * step + side, j0 = jt * FT;
    f32_wait_loads();
    W::publish();  // this step's tiles are in LDS; everyone is done with the other stage
    if (NST == 2 && step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    if (jt >= ntile || j0 > q0w + 31) continue;
    f32x16 s = f32_scores<DP>(tile(cur, side, 0), qf, lane);
    if (j0 + FT - 1 > q0w) {  // wave-uniform: only the tiles on the diagonal
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + f32_acc_row(v, hh) > q) s[v] = -INFINITY;
    }
    float mraw = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mraw = fmaxf(mraw, s[v]);
    float mx = fmaxf(m, mraw * sc2);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float alpha = __builtin_amdgcn_exp2f(m - mx);
    m = mx;
    l *= alpha;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], sc2, -mx));
      l += s[v];
    }
    f32_accumulate<DP>(tile(cur, side, 1), cb, s, o);
    if (NST == 1 && step + 1 < nstep) {
      W::publish();
      issue_step(step + 1, 0);
    }
  }
  f32_wait_loads();
  __syncthreads();
  float *x = reinterpret_cast<float *>(smem) + (size_t)grp * (SIDES - 1) * (DP / 2 + 2) * 64;  // [side][o..., m, l][lane]
  if (side > 0) {
    float *xs = SIDES == 2 ? x : x + (side - 1) * (DP / 2 + 2) * 64;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) xs[(dt * 16 + v) * 64 + lane] = o[dt][v];
    xs[(DP / 2) * 64 + lane] = m;
    xs[(DP / 2 + 1) * 64 + lane] = l;
  }
  __syncthreads();
  if (side == 0) {
    float mm = m;  // finite: the first side always has key tile 0
#pragma unroll
    for (int t = 0; t < SIDES - 1; ++t) mm = fmaxf(mm, x[(t * (DP / 2 + 2) + DP / 2) * 64 + lane]);
    const float a1 = __builtin_amdgcn_exp2f(m - mm);
    l *= a1;
#pragma unroll
    for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[dt][v] *= a1;
#pragma unroll
    for (int t = 0; t < SIDES - 1; ++t) {
      const float *xs = x + t * (DP / 2 + 2) * 64;
      const float a2 = __builtin_amdgcn_exp2f(xs[(DP / 2) * 64 + lane] - mm);
      l += xs[(DP / 2 + 1) * 64 + lane] * a2;
#pragma unroll
      for (int dt = 0; dt < DP / 32; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] += xs[(dt * 16 + v) * 64 + lane] * a2;
    }
    l += __shfl_xor(l, 32, 64);
    const uint32_t redo = nonfinite_rows(nonfinite_trace(o, l * 0.f), q < p.seq);  // see attn_rows.h
    if (q < p.seq && !((redo >> l32) & 1)) {
      f32_store<DP>(o, 1.f / l, p.ctx + ((int64_t)q * p.batch + n) * (p.nq * d) + g * d, d, hh);
      if (hh == 0) p.lse[((int64_t)n * p.nq + g) * p.seq + q] = row_lse(mm, l);
    }
    for (uint32_t r = redo; r; r &= r - 1) attn_row_fwd<float>(p, q0w + __builtin_ctz(r), g, n, lane);
  }
}

// ---- dQ: the same walk; dQ^T += K^T dS^T ----------------------------------------------------------------
template <int DP, int SIDES> __device__ __forceinline__ void f32_dq_block(const F32Params &p, char *smem, int qt, int g, int n) {
  using F = F32Tile<DP>;
  using W = F32Walk<DP, SIDES>;
  constexpr int FB = W::FB, NST = W::NST;
  const int kap = g / (p.nq / p.nkv), d = p.d;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave % W::GROUPS, side = wave / W::GROUPS, l32 = lane & 31, hh = lane >> 5;
  const int q0w = qt * FB + grp * 32, q = q0w + l32;
  const int64_t ts = (int64_t)p.batch * p.row, cs = (int64_t)p.batch * p.nq * d;
  const int koff = (p.nq + kap) * d, voff = (p.nq + p.nkv + kap) * d;
  const rsrc_t rs = make_rsrc(p.qkv, p.qkv_bytes);
  F32Loader<DP> ld;
  ld.init(ts, d, lane);
  auto tile = [&](int stage, int s, int which) { return smem + ((stage * SIDES + s) * 2 + which) * F::BYTES; };
  const bool valid = q < p.seq;
  f32x4 qf[DP / 8], dof[DP / 8];
  f32_row_frags<DP>(p.qkv + (int64_t)n * p.row + (int64_t)q * ts + g * d, valid, d, hh, qf);
  f32_row_frags<DP>(p.dctx + (int64_t)n * p.nq * d + (int64_t)q * cs + g * d, valid, d, hh, dof);
  const int64_t si = ((int64_t)n * p.nq + g) * p.seq + q;
  const float lse = valid ? p.lse_in[si] : 0.f, dvec = valid ? p.dvec[si] : 0.f;
  f32x16 acc[DP / 32];
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt) acc[dt] = f32_zero();
  const uint32_t cb = f32_cols_base<DP>(lane);
  const int kv_end = qt * FB + FB < p.seq ? qt * FB + FB : p.seq;
  const int ntile = (kv_end + FT - 1) / FT, nstep = (ntile + SIDES - 1) / SIDES;
  auto issue_step = [&](int step, int stage) {
    if constexpr (SIDES == 2) {
      const int s = wave >> 1, which = wave & 1, jt = 2 * step + s;
      if (jt < ntile) ld.issue(rs, tile(stage, s, which), (int64_t)jt * FT * ts, (int64_t)n * p.row + (which ? voff : koff));
    } else {
      const int jt = SIDES * step + side;
      if (jt < ntile) {
        ld.issue(rs, tile(stage, side, 0), (int64_t)jt * FT * ts, (int64_t)n * p.row + koff);
        ld.issue(rs, tile(stage, side, 1), (int64_t)jt * FT * ts, (int64_t)n * p.row + voff);
      }
    }
  };
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int cur = NST == 2 ? step & 1 : 0, jt = SIDES * step + side, j0 = jt * FT;
    f32_wait_loads();
    W::publish();
    if (NST == 2 && step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    if (jt >= ntile || j0 > q0w + 31) continue;
    f32x16 s = f32_scores<DP>(tile(cur, side, 0), qf, lane);
    const f32x16 dp = f32_scores<DP>(tile(cur, side, 1), dof, lane);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      s[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], p.scale, -lse) * kLog2ef) * (dp[v] - dvec);
    if (j0 + FT - 1 > q0w) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + f32_acc_row(v, hh) > q) s[v] = 0.f;
    }
    f32_accumulate<DP>(tile(cur, side, 0), cb, s, acc);
    if (NST == 1 && step + 1 < nstep) {
      W::publish();
      issue_step(step + 1, 0);
    }
  }
  f32_wait_loads();
  f32_join<DP, SIDES>(acc, reinterpret_cast<float *>(smem) + (size_t)grp * (SIDES - 1) * (DP / 2) * 64, side, lane);
  if (side > 0) return;
  const uint32_t redo = nonfinite_rows(nonfinite_trace(acc, 0.f), valid);  // see attn_rows.h
  if (valid && !((redo >> l32) & 1)) f32_store<DP>(acc, p.scale, p.dqkv + ((int64_t)q * p.batch + n) * p.row + g * d, d, hh);
  for (uint32_t r = redo; r; r &= r - 1) attn_row_dq<float>(p, q0w + __builtin_ctz(r), g, n, lane);
}

// ---- dK, dV: block = FB key rows of one (batch entry, query head); the sides take alternate query tiles -----------
template <int DP, int SIDES> __device__ __forceinline__ void f32_dkv_block(const F32Params &p, char *smem, int kt, int g, int n) {
  using F = F32Tile<DP>;
  using W = F32Walk<DP, SIDES>;
  constexpr int FB = W::FB, NST = W::NST;
  const int kap = g / (p.nq / p.nkv), d = p.d;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave % W::GROUPS, side = wave / W::GROUPS, l32 = lane & 31, hh = lane >> 5;
  const int j0w = kt * FB + grp * 32, j = j0w + l32;
  const int64_t ts = (int64_t)p.batch * p.row, cs = (int64_t)p.batch * p.nq * d;
  const int koff = (p.nq + kap) * d, voff = (p.nq + p.nkv + kap) * d;
  // SIDES = 2: the tile this wave fetches, Q or dO of a side
  const int my_side = SIDES == 2 ? wave >> 1 : side, my_which = SIDES == 2 ? wave & 1 : 0;
  const rsrc_t rs = my_which ? make_rsrc(p.dctx, p.ctx_bytes) : make_rsrc(p.qkv, p.qkv_bytes);
  F32Loader<DP> ld;
  ld.init(my_which ? cs : ts, d, lane);
  const rsrc_t rs_do = make_rsrc(p.dctx, p.ctx_bytes);
  F32Loader<DP> ld_do;  // SIDES = 4: a wave fetches both of its side
  if constexpr (SIDES == 4) ld_do.init(cs, d, lane);
  auto tile = [&](int stage, int s, int which) { return smem + ((stage * SIDES + s) * 2 + which) * F::BYTES; };
  float *stats = reinterpret_cast<float *>(smem + W::TILES);  // [stage][side][lse, D][32]
  const bool valid = j < p.seq;
  f32x4 kf[DP / 8], vf[DP / 8];
  f32_row_frags<DP>(p.qkv + (int64_t)n * p.row + (int64_t)j * ts + koff, valid, d, hh, kf);
  f32_row_frags<DP>(p.qkv + (int64_t)n * p.row + (int64_t)j * ts + voff, valid, d, hh, vf);
  f32x16 dk[DP / 32], dv[DP / 32];
#pragma unroll
  for (int dt = 0; dt < DP / 32; ++dt) dk[dt] = dv[dt] = f32_zero();
  const uint32_t cb = f32_cols_base<DP>(lane);
  const int it0 = kt * FB / FT, ntile = (p.seq + FT - 1) / FT - it0, nstep = (ntile + SIDES - 1) / SIDES;
  // the row statistics of a step are fetched one step ahead and put into LDS before the barrier that publishes its tiles:
  // SIDES = 2: wave 2 s holds lse, wave 2 s + 1 holds D of side s, lanes 0..31; SIDES = 4: the halves of a wave hold them
  float st = 0.f;
  auto issue_step = [&](int step, int stage) {
    const int it = SIDES * step + my_side, i0 = (it0 + it) * FT;
    st = 0.f;
    if (it < ntile) {
      ld.issue(rs, tile(stage, my_side, my_which), (int64_t)i0 * (my_which ? cs : ts),
               my_which ? (int64_t)n * p.nq * d + g * d : (int64_t)n * p.row + g * d);
      if constexpr (SIDES == 4) ld_do.issue(rs_do, tile(stage, my_side, 1), (int64_t)i0 * cs, (int64_t)n * p.nq * d + g * d);
      const int i = i0 + l32;
      if (i < p.seq) st = ((SIDES == 2 ? my_which : hh) ? p.dvec : p.lse_in)[((int64_t)n * p.nq + g) * p.seq + i];
    }
  };
  issue_step(0, 0);
  for (int step = 0; step < nstep; ++step) {
    const int cur = NST == 2 ? step & 1 : 0, it = SIDES * step + side, i0 = (it0 + it) * FT;
    f32_wait_loads();
    if (SIDES == 4 || lane < 32) stats[((cur * SIDES + my_side) * 2 + my_which) * FT + lane] = st;
    W::publish();
    if (NST == 2 && step + 1 < nstep) issue_step(step + 1, cur ^ 1);
    if (it >= ntile || i0 + 31 < j0w) continue;  // every query of the tile lies before every key of the wave
    const char *qt = tile(cur, side, 0), *dot = tile(cur, side, 1);
    const float *lse_s = stats + (cur * SIDES + side) * 2 * FT, *dv_s = lse_s + FT;
    f32x16 s = f32_scores<DP>(qt, kf, lane), dp = f32_scores<DP>(dot, vf, lane);
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 l4 = *reinterpret_cast<const f32x4 *>(lse_s + 8 * q4 + 4 * hh);
      const f32x4 d4 = *reinterpret_cast<const f32x4 *>(dv_s + 8 * q4 + 4 * hh);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = q4 * 4 + e;
        s[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], p.scale, -l4[e]) * kLog2ef);  // P
        dp[v] = s[v] * (dp[v] - d4[e]);                                                  // dS
      }
    }
    if (i0 < j0w + 31) {  // wave-uniform: only the tiles on the diagonal
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (i0 + f32_acc_row(v, hh) < j) s[v] = dp[v] = 0.f;
    }
    f32_accumulate<DP>(dot, cb, s, dv);
    f32_accumulate<DP>(qt, cb, dp, dk);
    if (NST == 1 && step + 1 < nstep) {
      W::publish();
      issue_step(step + 1, 0);
    }
  }
  f32_wait_loads();
  float *x = reinterpret_cast<float *>(smem) + (size_t)grp * (SIDES - 1) * (DP / 2) * 64;
  f32_join<DP, SIDES>(dk, x, side, lane);
  f32_join<DP, SIDES>(dv, x, side, lane);
  if (side > 0) return;
  const uint32_t redo = nonfinite_rows(nonfinite_trace(dk, nonfinite_trace(dv, 0.f)), valid);  // see attn_rows.h
  if (valid && !((redo >> l32) & 1)) {
    if (p.part) {
      float *out = p.part + (((int64_t)n * p.nq + g) * p.seq + j) * (2 * d);
      f32_store<DP>(dk, p.scale, out, d, hh);
      f32_store<DP>(dv, 1.f, out + d, d, hh);
    } else {
      float *out = p.dqkv + ((int64_t)j * p.batch + n) * p.row;
      f32_store<DP>(dk, p.scale, out + koff, d, hh);
      f32_store<DP>(dv, 1.f, out + voff, d, hh);
    }
  }
  for (uint32_t r = redo; r; r &= r - 1) attn_row_dkv<float>(p, j0w + __builtin_ctz(r), g, n, lane);
}

// Both halves of the backward pass in one launch: the dK/dV block of key tile r and the dQ block of query tile last - r
// alternate in dispatch order, both kinds longest walk first.
template <int DP, int SIDES> __global__ __launch_bounds__(256, 1) void f32_bwd_kernel(const F32Params p) {
  extern __shared__ __align__(1024) char smem[];
  const int rank = blockIdx.z >> 1, tiles = gridDim.z >> 1, g = blockIdx.x, n = blockIdx.y;
  if (blockIdx.z & 1) f32_dq_block<DP, SIDES>(p, smem, tiles - 1 - rank, g, n);
  else f32_dkv_block<DP, SIDES>(p, smem, rank, g, n);
}

// dK, dV of a kv head = sum of its query heads' partials, added in head order; thread = 4 columns
__global__ __launch_bounds__(256) void f32_dkv_reduce_kernel(const F32Params p) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // over [batch][nkv][seq][2 * d / 4]
  if (idx >= (int64_t)p.batch * p.nkv * p.seq * (2 * p.d / 4)) return;
  const int c4 = (int)(idx % (2 * p.d / 4));
  const int64_t r = idx / (2 * p.d / 4);
  const int j = (int)(r % p.seq);
  const int kap = (int)((r / p.seq) % p.nkv), n = (int)(r / ((int64_t)p.seq * p.nkv));
  const int group = p.nq / p.nkv;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int gg = 0; gg < group; ++gg)
    sum += *reinterpret_cast<const f32x4 *>(p.part + (((int64_t)n * p.nq + kap * group + gg) * p.seq + j) * (2 * p.d) + c4 * 4);
  const int which = c4 / (p.d / 4), col = (c4 % (p.d / 4)) * 4;  // 0: dK, 1: dV
  *reinterpret_cast<f32x4 *>(p.dqkv + ((int64_t)j * p.batch + n) * p.row + (p.nq + which * p.nkv + kap) * p.d + col) = sum;
}

// instantiated by name, ahead of the host code that takes their addresses
#define TM_F32_FAMILY(DP)                                          \
  template __global__ void f32_fwd_kernel<DP, 2>(const F32Params); \
  template __global__ void f32_bwd_kernel<DP, 2>(const F32Params); \
  template __global__ void f32_fwd_kernel<DP, 4>(const F32Params); \
  template __global__ void f32_bwd_kernel<DP, 4>(const F32Params);
TM_F32_FAMILY(32)
TM_F32_FAMILY(64)
TM_F32_FAMILY(96)
TM_F32_FAMILY(128)

// fp32 head sizes up to 128 of tensors that 32-bit offsets reach; the plain-ALU kernels take the rest
bool attn_f32_supported(int dtype, int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  return dtype == TM_DTYPE_FP32 && d <= 128 && seq * batch * (nq + 2 * nkv) * d * 4 < (1LL << 31);
}

static F32Params make_params(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d) {
  F32Params p = {};
  p.seq = (int)seq;
  p.batch = (int)batch;
  p.nq = (int)nq;
  p.nkv = (int)nkv;
  p.d = (int)d;
  p.row = (int)((nq + 2 * nkv) * d);
  p.scale = (float)(1.0 / sqrt((double)d));
  p.qkv_bytes = (uint32_t)(seq * batch * p.row * 4);
  p.ctx_bytes = (uint32_t)(seq * batch * nq * d * 4);
  return p;
}

// Four sides where a step's four tiles exist (a sequence of two is one step either way: 64 positions 6.9 / 6.9 us forward) and
// the chip has room: blocks of 32 rows fill a unit's LDS one at a time, so that up to 128 blocks of 64 rows (64 of each kind
// backward) stay one pass, and up to twice that two passes whose long and short walks even out from 256 positions.
// Two sides -> four, forward and backward, us: 128 positions, 8 walks of 64: 9.6 -> 7.1, 18.4 -> 14.0; 1024, 8: 47.8 -> 26.8,
// 83.7 -> 57.6; 512, 32 walks: 26.7 -> 21.6, 62.3 -> 68.7; 128, 128 walks: 10.4 -> 13.1, 26.9 -> 39.8; heads of 128, 512
// positions, 4 walks: 42.7 -> 26.5, 77.6 -> 49.5.  Four / two sides on 300 random calls (geometric mean): up to 128 blocks 0.76
// below 256 positions and 0.66 above, backward 0.81 and 0.70; 129 to 256 blocks of 256 positions and more 0.69 for heads of up to
// 64 and 0.74 above, with their one buffer (backward 0.75, 0.80), of fewer positions 1.0 (0.8 to 1.3).
static bool f32_four_sides(const F32Params &p, bool backward) {
  const int64_t blocks = ceil_div((int64_t)p.seq, (int64_t)64) * p.batch * p.nq * (backward ? 2 : 1);
  return p.seq > 64 && blocks <= (p.seq >= 256 ? 256 : 128);
}

template <int DP, int SIDES> static int launch_fwd(const F32Params &p, hipStream_t s) {
  using W = F32Walk<DP, SIDES>;
  static bool attr_set = false;  // per instantiation
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&f32_fwd_kernel<DP, SIDES>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       W::LDS) != hipSuccess)
    return fail(TM_ELAUNCH, "attn_fwd: cannot reserve LDS");
  attr_set = true;
  g_last_kernel = "f32_fwd_kernel";
  f32_fwd_kernel<DP, SIDES><<<dim3((unsigned)p.nq, (unsigned)p.batch, (unsigned)ceil_div(p.seq, W::FB)), 256, W::LDS, s>>>(p);
  return check_launch("attn_fwd_f32");
}
template <int DP> static int launch_fwd(const F32Params &p, hipStream_t s) {
  return f32_four_sides(p, false) ? launch_fwd<DP, 4>(p, s) : launch_fwd<DP, 2>(p, s);
}
template <int DP, int SIDES> static int launch_bwd(const F32Params &p, hipStream_t s) {
  using W = F32Walk<DP, SIDES>;
  static bool attr_set = false;
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&f32_bwd_kernel<DP, SIDES>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       W::LDS) != hipSuccess)
    return fail(TM_ELAUNCH, "attn_bwd: cannot reserve LDS");
  attr_set = true;
  g_last_kernel = "f32_bwd_kernel";
  f32_bwd_kernel<DP, SIDES><<<dim3((unsigned)p.nq, (unsigned)p.batch, 2 * (unsigned)ceil_div(p.seq, W::FB)), 256, W::LDS, s>>>(p);
  if (p.part) {
    const int64_t total = (int64_t)p.batch * p.nkv * p.seq * (2 * p.d / 4);
    f32_dkv_reduce_kernel<<<(unsigned)ceil_div(total, (int64_t)256), 256, 0, s>>>(p);
  }
  return check_launch("attn_bwd_f32");
}
template <int DP> static int launch_bwd(const F32Params &p, hipStream_t s) {
  return f32_four_sides(p, true) ? launch_bwd<DP, 4>(p, s) : launch_bwd<DP, 2>(p, s);
}

int attn_fwd_f32_launch(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d, const void *qkv, void *ctx, float *lse,
                        hipStream_t s) {
  F32Params p = make_params(seq, batch, nq, nkv, d);
  p.qkv = (const float *)qkv;
  p.ctx = (float *)ctx;
  p.lse = lse;
  if (d <= 32) return launch_fwd<32>(p, s);
  if (d <= 64) return launch_fwd<64>(p, s);
  if (d <= 96) return launch_fwd<96>(p, s);
  return launch_fwd<128>(p, s);
}

int attn_bwd_f32_launch(int64_t seq, int64_t batch, int64_t nq, int64_t nkv, int64_t d, const void *qkv, const void *dctx,
                        const float *lse, const float *dvec, float *part, void *dqkv, hipStream_t s) {
  F32Params p = make_params(seq, batch, nq, nkv, d);
  p.qkv = (const float *)qkv;
  p.dctx = (const float *)dctx;
  p.lse_in = lse;
  p.dvec = dvec;
  p.part = nq == nkv ? nullptr : part;
  p.dqkv = (float *)dqkv;
  if (d <= 32) return launch_bwd<32>(p, s);
  if (d <= 64) return launch_bwd<64>(p, s);
  if (d <= 96) return launch_bwd<96>(p, s);
  return launch_bwd<128>(p, s);
}

}  // namespace tmk
