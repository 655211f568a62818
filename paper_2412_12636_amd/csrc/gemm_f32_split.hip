// fp32 GEMM on the bf16 matrix instructions: every operand element as three bf16 terms.
//
// x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m: 24 significand bits in three times eight, exact as long as
// nothing underflows.  Of the nine products of two such sums the six down to 2^-16 of the largest are formed (hh, hm, mh, mm,
// hl, lh), the smallest first, into one fp32 accumulator; the three left out are below 2^-24 of |a b|, under the rounding
// of a fp32 product.  Six 32x32x16 MFMAs take 192 clocks where eight 32x32x2 fp32 ones take 512.
//
// A block has four waves that multiply and eight that fetch, four for each operand.  The fetching waves read fp32 rows from
// global memory two stages ahead into registers, split them (5.5 vector instructions an element) and write the three planes to
// LDS, [row][BK] bf16 each, for both kinds of layout: a lane that reads along a strided reduction axis holds a 4x4 block and
// packs its columns, which transposes it for free.  The multiplying waves own 64x64 results and read 16-byte fragments one
// batch of 24 MFMAs ahead.  Three LDS stages: one read, one complete (its first fragments are fetched ahead of the barrier), one
// written.  The results leave through LDS as whole rows, all twelve waves storing.
//
// 128x128 tiles: bound by the MFMA rate that random data sustains (1.13 us a stage of 32 elements with every unit busy and
// nothing to fetch or split, 0.9 with a quarter of them, 0.64 at the nominal clock); 1.24 to 1.3 measured, 1.2 PFLOP/s of bf16
// products = 200 TFLOP/s of fp32 ones.  64x64 tiles: a stage of 64 elements takes 0.9 us where its MFMAs take 0.35 to 0.6;
// splitting operands that serve only 64 results of the other side costs as much as multiplying them.  With four fetching waves
// instead of eight 1.0; with chunks placed for 32 LDS banks instead of 64 1.1; with results stored by the waves that hold them
// 2 us more a block.
// Against the fp32 instructions: 1024 x 8192 over 1024 131 -> 88 us, 1024 x 4096 over 1024 70 -> 47, 2048 x 2048 over 2048 142 -> 85,
// 1024 x 1024 over 1024 23.6 -> 17.5, over 4096 72 -> 57.
#include "gemm.h"
#include "gemm_f32_form.h"

namespace tmk {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int v4u32 __attribute__((__vector_size__(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitPatch = 8;  // row-tiles of a patch

struct F32SplitParams {
  int M, N, K;
  const float *A, *B;
  int64_t lda, ldb;  // the non-unit strides
  float *C;
  int64_t ldc;
  const float *bias, *residual;
  int tiles_m, tiles_n;
  uint32_t a_bytes, b_bytes, c_bytes;
};

// Byte of 16-byte chunk c of a row in a plane [R][BK].  Sixteen lanes that read one chunk of sixteen consecutive rows, and 32
// that write eight bytes each, of whole rows or of two chunks of eight rows four apart, meet each of the 64 banks once.
template <int BK> __device__ __forceinline__ int plane_pos(int row, int c) {
  if (BK == 32)
    return (row >> 2) * 256 + ((row ^ (row >> 2)) & 3) * 64 + ((c ^ ((row >> 2) & 3) ^ ((row >> 3) & 2)) << 4);
  return (row >> 1) * 256 + ((row ^ (row >> 2)) & 1) * 128 + ((c ^ ((row >> 2) & 3) ^ (((row >> 2) ^ (row << 1)) & 4)) << 4);
}

// The leading bf16 of both, and what it leaves.  (x - h as one bf16 dot product with -1, seven instructions for three terms of
// two elements instead of eleven, is exact too but shares the matrix cores: a stage of 128x128 tiles 0.92 -> 1.18 us.)
__device__ __forceinline__ uint32_t split_term(f32x2 &x) {
  const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
  x[0] -= __builtin_bit_cast(float, h << 16);
  x[1] -= __builtin_bit_cast(float, h & 0xffff0000u);
  return h;
}
template <int PLANE> __device__ __forceinline__ void write_terms(char *at, f32x2 x, f32x2 y) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const uint32_t a = split_term(x), b = split_term(y);
    *reinterpret_cast<u32x2 *>(at + p * PLANE) = u32x2{a, b};
  }
}

// Fetching four waves' share of R rows by BK reduction elements.
template <int R, int BK, bool KC> struct SplitLoad {
  static constexpr int PLANE = R * BK * 2, NL = R * BK / 1024;  // 16-byte loads of a lane
  uint32_t voff[NL];
  int k_first[NL], lds_at[NL];
  f32x4 x[2][NL];
  __device__ __forceinline__ void init(int64_t ld, int row0, int t) {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int idx = i * 256 + t, row = idx / (BK / 4), kc = idx % (BK / 4);
        voff[i] = (uint32_t)(((int64_t)(row0 + row) * ld + kc * 4) * 4);
        k_first[i] = kc * 4;
        lds_at[i] = plane_pos<BK>(row, kc >> 1) + (kc & 1) * 8;
      }
    } else {  // a wave: eight row groups by eight groups of four reduction elements; element i of the block is a load
      static_assert(NL == 4, "one block of 4x4 a lane");
      const int wave = t / 64, lane = t % 64;
      const int kg = wave % (BK / 32) * 8 + lane / 8, rg = wave / (BK / 32) * 8 + lane % 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        k_first[i] = kg * 4 + i;
        voff[i] = (uint32_t)(((int64_t)k_first[i] * ld + row0 + rg * 4) * 4);
        lds_at[i] = plane_pos<BK>(rg * 4 + i, kg >> 1) + (kg & 1) * 8;
      }
    }
  }
  // elements past the end of the reduction read outside the tensor (zero)
  template <int SET> __device__ __forceinline__ void fetch(rsrc_t rs, int k0, int K, int64_t ld) {
    const uint32_t koff = KC ? (uint32_t)k0 * 4u : (uint32_t)((int64_t)k0 * ld * 4);
#pragma unroll
    for (int i = 0; i < NL; ++i)
      x[SET][i] = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, k0 + k_first[i] < K ? voff[i] + koff : 0x80000000u, 0, 0));
  }
  template <int SET> __device__ __forceinline__ void store(char *tile) const {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if constexpr (KC)
        write_terms<PLANE>(tile + lds_at[i], f32x2{x[SET][i][0], x[SET][i][1]}, f32x2{x[SET][i][2], x[SET][i][3]});
      else
        write_terms<PLANE>(tile + lds_at[i], f32x2{x[SET][0][i], x[SET][1][i]}, f32x2{x[SET][2][i], x[SET][3][i]});
    }
  }
};

// A wave's LDS accesses are complete (lgkmcnt 0 as an instruction that the compiler counts with), then everyone's.
__device__ __forceinline__ void split_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The lane's number behind the main loop, without a register that holds it during the loop.
__device__ __forceinline__ int lane_again() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// The 32x32 results at (m0, n0) again on the fp32 matrix instructions, operands straight from global memory: for tiles with a
// value that is not finite (an infinite element has no remainder, one above the largest bf16 has an infinite leading term) or
// with an operand row of nothing but elements below 2^-95, whose lower terms the bf16 instructions take for zero.
template <bool A_KC, bool B_KC>
__device__ __forceinline__ f32x16 fp32_tile(const F32SplitParams &p, int m0, int n0, int lane) {
  const rsrc_t ra = make_rsrc(p.A, p.a_bytes), rb = make_rsrc(p.B, p.b_bytes);
  auto frag = [&](rsrc_t rs, bool kc, int64_t ld, int row, int rows, int k) {
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      x[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                 rs, row < rows && k + i < p.K ? (uint32_t)((kc ? row * ld + k + i : (k + i) * ld + row) * 4) : 0x80000000u, 0, 0));
    return x;
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int k0 = 0; k0 < p.K; k0 += 8) {
    const f32x4 a = frag(ra, A_KC, p.lda, m0 + lane % 32, p.M, k0 + 4 * (lane / 32));
    const f32x4 b = frag(rb, B_KC, p.ldb, n0 + lane % 32, p.N, k0 + 4 * (lane / 32));
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
  }
  return acc;
}

template <int BM, int BN, int BK> struct F32SplitCfg {
  static constexpr int NT = (BM / 64) * (BN / 64), KSPL = 4 / NT, SUBS = BK / 16 / KSPL;
  static constexpr int PA = BM * BK * 2, PB = BN * BK * 2, STAGE = 3 * (PA + PB);
  // the results of a wave's share of the reduction on their way out; 4 PITCH is 32 banks off a whole round of 64
  static constexpr int PITCH = BN + 8, OUT = BM * PITCH * 4, LDS = 3 * STAGE > KSPL * OUT ? 3 * STAGE : KSPL * OUT;
  static_assert(NT * KSPL == 4 && SUBS >= 1 && 4 * PITCH % 64 == 32, "four multiplying waves of 64x64");
};

template <int BM, int BN, int BK, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(768) void gemm_f32_split_kernel(const F32SplitParams p) {
  typedef F32SplitCfg<BM, BN, BK> C;
  constexpr int KSPL = C::KSPL, SUBS = C::SUBS, NT = C::NT;
  extern __shared__ __align__(1024) char lds[];
  // an XCD (ids round-robin over eight) owns a range of tiles, walked in patches
  const int nblk = p.tiles_m * p.tiles_n, xcd = blockIdx.x % 8, base = nblk / 8, rem = nblk % 8;
  const int lid = xcd * base + (xcd < rem ? xcd : rem) + (int)(blockIdx.x / 8);
  const int gi = lid / (kSplitPatch * p.tiles_n), first = gi * kSplitPatch, in_group = lid - first * p.tiles_n;
  const int rows = p.tiles_m - first < kSplitPatch ? p.tiles_m - first : kSplitPatch;
  const int m0 = (first + in_group % rows) * BM, n0 = (in_group / rows) * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nk = (p.K + BK - 1) / BK;
  float *const out = reinterpret_cast<float *>(lds);
  bool redo = false;

  if (wave >= 4) {
    auto feed = [&](auto load, const float *src, uint32_t bytes, int64_t ld, int row0, char *slot) {
      const rsrc_t rs = make_rsrc(src, bytes);
      char *const last = slot + 2 * C::STAGE;
      load.init(ld, row0, (int)threadIdx.x & 255);
      load.template fetch<0>(rs, 0, p.K, ld);
      if (nk > 1) load.template fetch<1>(rs, BK, p.K, ld);
      auto stage = [&](auto set, int s) {
        constexpr int SET = decltype(set)::value;
        load.template store<SET>(slot);
        if (s + 2 < nk) load.template fetch<SET>(rs, (s + 2) * BK, p.K, ld);
        slot = slot == last ? slot - 2 * C::STAGE : slot + C::STAGE;
        split_barrier();  // stage s is whole; stage s - 2 has been read
      };
      for (int s = 0; s < nk; s += 2) {
        stage(std::integral_constant<int, 0>{}, s);
        if (s + 1 < nk) stage(std::integral_constant<int, 1>{}, s + 1);
      }
    };
    if (wave < 8)
      feed(SplitLoad<BM, BK, A_KC>{}, p.A, p.a_bytes, p.lda, m0, lds);
    else
      feed(SplitLoad<BN, BK, B_KC>{}, p.B, p.b_bytes, p.ldb, n0, lds + 3 * C::PA);
    split_barrier();
    split_barrier();
  } else {
    const int ks = wave / NT, wt = wave % NT;
    const int wm = wt / (BN / 64) * 64, wn = wt % (BN / 64) * 64;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    struct Frags {
      bf16x8 a[2][3], b[2][3];
    } f[2];
    static_assert(SUBS <= 2, "the second 16 reduction elements of a wave: 32 bytes across in the lane address");
    const int at = plane_pos<BK>(lane % 32, 2 * ks * SUBS + lane / 32);
    auto fetch = [&](Frags &x, const char *slot, int s) {
      const char *A = slot + wm * BK * 2 + (at ^ (s * 32)), *B = slot + 3 * C::PA + wn * BK * 2 + (at ^ (s * 32));
#pragma unroll
      for (int q = 2; q >= 0; --q)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          x.a[t][q] = *reinterpret_cast<const bf16x8 *>(A + q * C::PA + t * 32 * BK * 2);
          x.b[t][q] = *reinterpret_cast<const bf16x8 *>(B + q * C::PB + t * 32 * BK * 2);
        }
    };
    uint32_t bits[4] = {0, 0, 0, 0};  // of the leading terms of the lane's rows: of A in both tiles, of B in both
    auto multiply = [&](const Frags &x) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const u32x4 a = __builtin_bit_cast(u32x4, x.a[t][0]), b = __builtin_bit_cast(u32x4, x.b[t][0]);
        bits[t] |= a[0] | a[1], bits[t] |= a[2] | a[3];
        bits[2 + t] |= b[0] | b[1], bits[2 + t] |= b[2] | b[3];
      }
      constexpr int qa[6] = {2, 0, 1, 1, 0, 0}, qb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
          for (int tn = 0; tn < 2; ++tn)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[tm][qa[q]], x.b[tn][qb[q]], acc[tm][tn], 0, 0, 0);
    };
    const char *cur = lds, *next = lds + C::STAGE;
    auto advance = [&] {
      cur = next;
      next = next == lds + 2 * C::STAGE ? lds : next + C::STAGE;
    };
    split_barrier();
    fetch(f[0], cur, 0);
    if constexpr (SUBS == 1) {
      for (int t = 0; t < nk; t += 2) {  // (the fragments fetched behind the last stage are not used)
        split_barrier();
        fetch(f[1], next, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f[0]);
        advance();
        if (t + 1 < nk) {
          split_barrier();
          fetch(f[0], next, 0);
          __builtin_amdgcn_sched_barrier(0);
          multiply(f[1]);
          advance();
        }
      }
    } else {
      static_assert(SUBS == 1 || SUBS % 2 == 0, "fragment sets alternate");
      for (int t = 0; t < nk; ++t) {
        split_barrier();
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
          fetch(f[(s + 1) & 1], s + 1 < SUBS ? cur : next, (s + 1) % SUBS);
          __builtin_amdgcn_sched_barrier(0);
          multiply(f[s & 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
        advance();
      }
    }

    const int out_lane = lane_again();
    split_barrier();  // everyone has read its last fragments
    float *x = out + ks * (C::OUT / 4) + (wm + 4 * (out_lane >> 5)) * C::PITCH + wn + out_lane % 32;
    float finite = 0.f;  // stays zero unless a product with an infinity or NaN gets in
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float r = acc[i >> 1][i & 1][v];
        x[((i >> 1) * 32 + 8 * (v >> 2) + (v & 3)) * C::PITCH + (i & 1) * 32] = r;
        finite = __builtin_fmaf(r, 0.f, finite);
      }
    redo = finite != 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {  // all of a row's elements below 2^-95 (an exponent field under 32), and not all zero
      const uint32_t b = bits[t] | (uint32_t)__shfl_xor((int)bits[t], 32), e = b | b >> 16;
      redo |= (e & 0x7fff) != 0 && (e & 0x7000) == 0;
    }
  }
  const int out_lane = lane_again(), tid = wave * 64 + out_lane;
  if (__syncthreads_or(redo)) {
    for (int i = wave; i < (BM / 32) * (BN / 32); i += 12) {
      const int tm = i / (BN / 32) * 32, tn = i % (BN / 32) * 32;
      const f32x16 r = fp32_tile<A_KC, B_KC>(p, m0 + tm, n0 + tn, out_lane);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float *x = out + (tm + 8 * (v >> 2) + 4 * (out_lane >> 5) + (v & 3)) * C::PITCH + tn + out_lane % 32;
        x[0] = r[v];
        for (int w = 1; w < KSPL; ++w) x[w * (C::OUT / 4)] = 0.f;
      }
    }
    __syncthreads();
  }
  const rsrc_t rc = make_rsrc(p.C, p.c_bytes), rres = make_rsrc(p.residual, p.c_bytes);
  const int col = tid % (BN / 4) * 4;
  f32x4 bias = {0.f, 0.f, 0.f, 0.f};
  if (EPI == 0 && p.bias && n0 + col < p.N) bias = *reinterpret_cast<const f32x4 *>(p.bias + n0 + col);
#pragma unroll 2
  for (int row = tid / (BN / 4); row < BM; row += 768 / (BN / 4)) {
    const float *x = out + row * C::PITCH + col;
    f32x4 r = *reinterpret_cast<const f32x4 *>(x);
#pragma unroll
    for (int w = 1; w < KSPL; ++w) r += *reinterpret_cast<const f32x4 *>(x + w * (C::OUT / 4));
    const uint32_t off = m0 + row < p.M && n0 + col < p.N ? (uint32_t)(((int64_t)(m0 + row) * p.ldc + n0 + col) * 4) : 0x80000000u;
    if (EPI == 0) {
      r += bias;
      if (p.residual) r += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rres, off, 0, 0));
    } else if (EPI == 1) {
      r += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, off, 0, 0));
    }
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u32, r), rc, off, 0, 0);
  }
}

template <int BM, int BN, int BK, bool A_KC, bool B_KC, int EPI> static int launch(const GemmArgs &g, hipStream_t s) {
  F32SplitParams p;
  p.M = (int)g.M;
  p.N = (int)g.N;
  p.K = (int)g.K;
  p.A = (const float *)g.A;
  p.lda = A_KC ? g.a_rs : g.a_cs;
  p.B = (const float *)g.B;
  p.ldb = B_KC ? g.b_rs : g.b_cs;
  p.C = (float *)g.C;
  p.ldc = g.ldc;
  p.bias = (const float *)g.bias;
  p.residual = (const float *)g.residual;
  p.tiles_m = (int)ceil_div(g.M, BM);
  p.tiles_n = (int)ceil_div(g.N, BN);
  p.a_bytes = (uint32_t)((A_KC ? g.M * g.a_rs : g.K * g.a_cs) * 4);
  p.b_bytes = (uint32_t)((B_KC ? g.N * g.b_rs : g.K * g.b_cs) * 4);
  p.c_bytes = (uint32_t)(g.M * g.ldc * 4);
  constexpr int lds = F32SplitCfg<BM, BN, BK>::LDS;
  static bool attr_set = false;  // per instantiation
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_f32_split_kernel<BM, BN, BK, A_KC, B_KC, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
    return fail(TM_ELAUNCH, "gemm_f32_split: cannot reserve %d bytes of LDS", lds);
  attr_set = true;
  const int64_t blocks = (int64_t)p.tiles_m * p.tiles_n;
  if (blocks > 0x7fffffff) return fail(TM_ESIZE, "gemm_f32_split: too many tiles");
  g_last_kernel = "gemm_f32_split_kernel";
  gemm_f32_split_kernel<BM, BN, BK, A_KC, B_KC, EPI><<<(unsigned)blocks, 768, lds, s>>>(p);
  return check_launch("gemm_f32_split");
}

template <bool A_KC, bool B_KC, int EPI> static int pick(const GemmArgs &g, int tile, hipStream_t s) {
  if (tile == 128) return launch<128, 128, 32, A_KC, B_KC, EPI>(g, s);
  return launch<64, 64, 64, A_KC, B_KC, EPI>(g, s);
}

bool gemm_f32_split_supported(const GemmArgs &g) {
  return gemm_f32_supported(g) && g.N % 4 == 0 && g.ldc % 4 == 0 && (((uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.residual) & 15) == 0;
}

int gemm_f32_split(const GemmArgs &g, int tile, hipStream_t s) {
  if (g.c_mode == 1) return pick<false, false, 1>(g, tile, s);
  if (g.c_mode == 2) return pick<false, false, 2>(g, tile, s);
  return g.b_cs == 1 ? pick<true, true, 0>(g, tile, s) : pick<true, false, 0>(g, tile, s);
}

}  // namespace tmk
