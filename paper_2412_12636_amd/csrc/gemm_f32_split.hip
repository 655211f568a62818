// fp32 GEMM on the bf16 matrix instructions: every operand element as three bf16 terms.
//
// 2^24 x = h + m + l with h = bf16(2^24 x), m = bf16 of what h leaves, l the rest: 24 significand bits in three times eight.
// The instructions take subnormal terms for zero; at this scale the last bit of any x is 2^-125 or more, so that no term is
// subnormal and the sum is exact, small elements beside large ones included.  Elements of 2^104 and more and results of 2^80
// and more come out as infinities and NaN, and are formed on the fp32 instructions as those are.  Of the nine products of two
// such sums all but ll are formed, which is below 2^-34 of |a b|.  hh is exact in fp32 and has an accumulator of its own; the
// seven others, 2^-8 of it and less, share a second one, and the two meet once at the end.  What rounds is one sum of hh for
// every eight elements, where a chain of fused multiply-adds rounds each.  Errors against 64 bits, of the result, fp32
// instructions / here: 256 N(0,1) elements 2.9e-7 / 0.9e-7, 2048 8.1e-7 / 2.7e-7; rows of 16 elements that are not zero 7.4e-8
// / 3.4e-8, of four 4.0e-8 / 2.6e-8, of one 2.53e-8 / 2.53e-8 (0.500 / 0.506 ulp at most).  With all terms in one accumulator
// these were 1.4e-7, 7.3e-8 and 3.5e-8 (1.4 ulp); with ml and lm left out 3.4e-8, 2.7e-8 and 2.6e-8 (0.95 ulp).
// Eight 32x32x16 MFMAs take 256 clocks where eight 32x32x2 fp32 ones take 512.
//
// A block has four waves that multiply and four that fetch, two for each operand.  The fetching waves read fp32 rows from
// global memory two stages ahead into registers, split them (6.5 vector instructions an element) and write the three planes to
// LDS, [row][32] bf16 each, for both kinds of layout: a lane that reads along a strided reduction axis holds 4x4 blocks and
// packs their columns, which transposes them for free.  The multiplying waves own 64x64 results and read 16-byte fragments one
// batch of 32 MFMAs ahead; two sets of fragments and two of accumulators are 224 of the 256 registers that two waves a SIMD
// leave.  Three LDS stages: one read, one complete (its first fragments are fetched ahead of the barrier), one written.  The
// results leave through LDS as whole rows, all eight waves storing.
//
// Bound by the MFMA rate that random data sustains: a stage of 32 elements takes 1.43 us with every unit busy (188 TFLOP/s of fp32
// products), 1.5 at that rate and 0.85 at the nominal clock; the matrix cores are busy for 65 to 68 % of the cycles, first loads and
// epilogue included.  Neither a higher priority of the fetching or the multiplying waves nor fewer scheduling barriers change it by
// more than 2 %.  64x64 tiles, whose operands are split for only 64 results of the other side, were 6 % slower than the fp32
// instructions (1024 x 1024 over 1024 21.6 us against 20.4).
// Against the fp32 instructions: 1024 x 8192 over 1024 137 -> 114 us, 1024 x 4096 over 1024 77 -> 58, 2048 x 2048 over 2048 135 -> 108.
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

constexpr int kSplitPatch = 8;  // row-tiles of a patch
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;  // the operands' scale, and back from their products'

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

constexpr int kTile = 128, kStep = 32;            // a block's results; reduction elements of a stage
constexpr int kPlane = kTile * kStep * 2;         // a term of an operand's stage, [row][kStep] bf16
constexpr int kStage = 6 * kPlane, kStages = 3;   // A's terms, B's terms
constexpr int kOutPitch = kTile + 8;              // floats; 4 of these are 32 banks off a whole round of 64
constexpr int kSplitLds = kStages * kStage;
static_assert(kTile * kOutPitch * 4 <= kSplitLds, "the results leave through the stages' place");

// Byte of 16-byte chunk c of a row in a plane.  Sixteen lanes that read one chunk of sixteen consecutive rows, and 32 that write
// eight bytes each, of whole rows or of two chunks of eight rows four apart, meet each of the 64 banks once.
__device__ __forceinline__ int plane_pos(int row, int c) {
  return (row >> 2) * 256 + ((row ^ (row >> 2)) & 3) * 64 + ((c ^ ((row >> 2) & 3) ^ ((row >> 3) & 2)) << 4);
}

// The leading bf16 of both, and what it leaves.  (x - h as one bf16 dot product with -1, seven instructions for three terms of
// two elements instead of eleven, is exact too but shares the matrix cores: a stage of 128x128 tiles 0.92 -> 1.18 us.)
__device__ __forceinline__ uint32_t split_term(f32x2 &x) {
  const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
  x[0] -= __builtin_bit_cast(float, h << 16);
  x[1] -= __builtin_bit_cast(float, h & 0xffff0000u);
  return h;
}
__device__ __forceinline__ void write_terms(char *at, f32x2 x, f32x2 y) {
  x[0] *= kUp, x[1] *= kUp, y[0] *= kUp, y[1] *= kUp;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const uint32_t a = split_term(x), b = split_term(y);
    *reinterpret_cast<u32x2 *>(at + p * kPlane) = u32x2{a, b};
  }
}

// Fetching two waves' share of a stage of one operand.
template <bool KC> struct SplitLoad {
  static constexpr int NL = kTile * kStep / 512;  // 16-byte loads of a lane
  uint32_t voff[NL];
  int k_first[NL], lds_at[NL];
  f32x4 x[2][NL];
  __device__ __forceinline__ void init(int64_t ld, int row0, int t) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if constexpr (KC) {
        const int idx = i * 128 + t, row = idx / (kStep / 4), kc = idx % (kStep / 4);
        voff[i] = (uint32_t)(((int64_t)(row0 + row) * ld + kc * 4) * 4);
        k_first[i] = kc * 4;
        lds_at[i] = plane_pos(row, kc >> 1) + (kc & 1) * 8;
      } else {  // a wave, twice: eight row groups by eight groups of four reduction elements; element i % 4 of a block is a load
        const int kg = t % 64 / 8, rg = (t / 64 + i / 4 * 2) * 8 + t % 8;
        k_first[i] = kg * 4 + i % 4;
        voff[i] = (uint32_t)(((int64_t)k_first[i] * ld + row0 + rg * 4) * 4);
        lds_at[i] = plane_pos(rg * 4 + i % 4, kg >> 1) + (kg & 1) * 8;
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
      const f32x4 *b = x[SET] + i / 4 * 4;
      if constexpr (KC)
        write_terms(tile + lds_at[i], f32x2{x[SET][i][0], x[SET][i][1]}, f32x2{x[SET][i][2], x[SET][i][3]});
      else
        write_terms(tile + lds_at[i], f32x2{b[0][i % 4], b[1][i % 4]}, f32x2{b[2][i % 4], b[3][i % 4]});
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
// value that is not finite (an infinite element has no remainder, one that the scale takes past the largest bf16 has an infinite
// leading term).  Bound by the loads' latency, hence 16 of them under way: 2048 x 2048 over 2048 110 us, with an infinite row 160
// (weight gradient 310), all of it formed again 280 to 315, 130 to 157 on the fp32 instructions alone; with one load of four
// under way at a time all of it took 420 to 970.
template <bool A_KC, bool B_KC>
__device__ __forceinline__ f32x16 fp32_tile(const F32SplitParams &p, int m0, int n0, int lane) {
  const rsrc_t ra = make_rsrc(p.A, p.a_bytes), rb = make_rsrc(p.B, p.b_bytes);
  auto frag = [&](auto kc, rsrc_t rs, int64_t ld, int row, int rows, int k) {  // four reduction elements (K: a multiple of 4 if kc)
    f32x4 x;
    if constexpr (decltype(kc)::value) {
      x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
              rs, row < rows && k < p.K ? (uint32_t)((row * ld + k) * 4) : 0x80000000u, 0, 0));
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        x[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                   rs, row < rows && k + i < p.K ? (uint32_t)(((k + i) * ld + row) * 4) : 0x80000000u, 0, 0));
    }
    return x;
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  constexpr int kAhead = 8;  // loads of both operands under way, eight elements each
  for (int k0 = 0; k0 < p.K; k0 += 8 * kAhead) {
    f32x4 a[kAhead], b[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k = k0 + 8 * j + 4 * (lane / 32);
      a[j] = frag(std::bool_constant<A_KC>{}, ra, p.lda, m0 + lane % 32, p.M, k);
      b[j] = frag(std::bool_constant<B_KC>{}, rb, p.ldb, n0 + lane % 32, p.N, k);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j][i], b[j][i], acc, 0, 0, 0);
  }
  return acc;
}

template <bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(512) void gemm_f32_split_kernel(const F32SplitParams p) {
  extern __shared__ __align__(1024) char lds[];
  // an XCD (ids round-robin over eight) owns a range of tiles, walked in patches
  const int nblk = p.tiles_m * p.tiles_n, xcd = blockIdx.x % 8, base = nblk / 8, rem = nblk % 8;
  const int lid = xcd * base + (xcd < rem ? xcd : rem) + (int)(blockIdx.x / 8);
  const int gi = lid / (kSplitPatch * p.tiles_n), first = gi * kSplitPatch, in_group = lid - first * p.tiles_n;
  const int rows = p.tiles_m - first < kSplitPatch ? p.tiles_m - first : kSplitPatch;
  const int m0 = (first + in_group % rows) * kTile, n0 = (in_group / rows) * kTile;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nk = (p.K + kStep - 1) / kStep;
  float *const out = reinterpret_cast<float *>(lds);
  bool redo = false;

  if (wave >= 4) {
    auto feed = [&](auto load, const float *src, uint32_t bytes, int64_t ld, int row0, char *slot) {
      const rsrc_t rs = make_rsrc(src, bytes);
      char *const last = slot + (kStages - 1) * kStage;
      load.init(ld, row0, (int)threadIdx.x & 127);
      load.template fetch<0>(rs, 0, p.K, ld);
      if (nk > 1) load.template fetch<1>(rs, kStep, p.K, ld);
      auto stage = [&](auto set, int s) {
        constexpr int SET = decltype(set)::value;
        load.template store<SET>(slot);
        if (s + 2 < nk) load.template fetch<SET>(rs, (s + 2) * kStep, p.K, ld);
        slot = slot == last ? slot - (kStages - 1) * kStage : slot + kStage;
        split_barrier();  // stage s is whole; stage s - 2 has been read
      };
      for (int s = 0; s < nk; s += 2) {
        stage(std::integral_constant<int, 0>{}, s);
        if (s + 1 < nk) stage(std::integral_constant<int, 1>{}, s + 1);
      }
    };
    if (wave < 6)
      feed(SplitLoad<A_KC>{}, p.A, p.a_bytes, p.lda, m0, lds);
    else
      feed(SplitLoad<B_KC>{}, p.B, p.b_bytes, p.ldb, n0, lds + 3 * kPlane);
    split_barrier();
    split_barrier();
  } else {
    const int wm = wave / 2 * 64, wn = wave % 2 * 64;
    f32x16 lead[2][2], rest[2][2];  // the leading terms' products; all others
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) lead[i >> 1][i & 1][v] = rest[i >> 1][i & 1][v] = 0.f;
    struct Frags {
      bf16x8 a[2][3], b[2][3];
    } f[2];
    const int at = plane_pos(lane % 32, lane / 32);  // (the second 16 reduction elements: 32 bytes across)
    auto fetch = [&](Frags &x, const char *slot, int s) {
      const char *A = slot + wm * kStep * 2 + (at ^ (s * 32)), *B = slot + 3 * kPlane + wn * kStep * 2 + (at ^ (s * 32));
#pragma unroll
      for (int q = 2; q >= 0; --q)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          x.a[t][q] = *reinterpret_cast<const bf16x8 *>(A + q * kPlane + t * 32 * kStep * 2);
          x.b[t][q] = *reinterpret_cast<const bf16x8 *>(B + q * kPlane + t * 32 * kStep * 2);
        }
    };
    auto multiply = [&](const Frags &x) {
      constexpr int qa[8] = {0, 2, 1, 2, 0, 1, 1, 0}, qb[8] = {0, 1, 2, 0, 2, 1, 0, 1};
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f32x16 &to = q ? rest[i >> 1][i & 1] : lead[i >> 1][i & 1];
          to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[i >> 1][qa[q]], x.b[i & 1][qb[q]], to, 0, 0, 0);
        }
    };
    const char *cur = lds, *next = lds + kStage;
    split_barrier();
    fetch(f[0], cur, 0);
    for (int t = 0; t < nk; ++t) {
      split_barrier();
      fetch(f[1], cur, 1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(f[0]);
      __builtin_amdgcn_sched_barrier(0);
      fetch(f[0], next, 0);  // (behind the last stage: not used)
      __builtin_amdgcn_sched_barrier(0);
      multiply(f[1]);
      __builtin_amdgcn_sched_barrier(0);
      cur = next;
      next = next == lds + (kStages - 1) * kStage ? lds : next + kStage;
    }

    const int out_lane = lane_again();
    split_barrier();  // everyone has read its last fragments
    float *x = out + (wm + 4 * (out_lane >> 5)) * kOutPitch + wn + out_lane % 32;
    float finite = 0.f;  // stays zero unless a product with an infinity or NaN gets in
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float r = (lead[i >> 1][i & 1][v] + rest[i >> 1][i & 1][v]) * kDown;
        x[((i >> 1) * 32 + 8 * (v >> 2) + (v & 3)) * kOutPitch + (i & 1) * 32] = r;
        finite = __builtin_fmaf(r, 0.f, finite);
      }
    redo = finite != 0.f;
  }
  const int out_lane = lane_again(), tid = wave * 64 + out_lane;
  if (__syncthreads_or(redo)) {
    // only results that are not finite are replaced, so that no row's bits depend on what the others hold
    for (int i = wave; i < 16; i += 8) {
      const int tm = i / 4 * 32, tn = i % 4 * 32;
      float *x = out + (tm + 4 * (out_lane >> 5)) * kOutPitch + tn + out_lane % 32;
      bool bad = false;
#pragma unroll
      for (int v = 0; v < 16; ++v) bad |= !__builtin_isfinite(x[(8 * (v >> 2) + (v & 3)) * kOutPitch]);
      if (!__any(bad)) continue;
      const f32x16 r = fp32_tile<A_KC, B_KC>(p, m0 + tm, n0 + tn, out_lane);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float &at = x[(8 * (v >> 2) + (v & 3)) * kOutPitch];
        if (!__builtin_isfinite(at)) at = r[v];
      }
    }
    __syncthreads();
  }
  const rsrc_t rc = make_rsrc(p.C, p.c_bytes), rres = make_rsrc(p.residual, p.c_bytes);
  const int col = tid % (kTile / 4) * 4;
  f32x4 bias = {0.f, 0.f, 0.f, 0.f};
  if (EPI == 0 && p.bias && n0 + col < p.N) bias = *reinterpret_cast<const f32x4 *>(p.bias + n0 + col);
#pragma unroll 2
  for (int row = tid / (kTile / 4); row < kTile; row += 512 / (kTile / 4)) {
    f32x4 r = *reinterpret_cast<const f32x4 *>(out + row * kOutPitch + col);
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

template <bool A_KC, bool B_KC, int EPI> static int launch(const GemmArgs &g, hipStream_t s) {
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
  p.tiles_m = (int)ceil_div(g.M, kTile);
  p.tiles_n = (int)ceil_div(g.N, kTile);
  p.a_bytes = (uint32_t)((A_KC ? g.M * g.a_rs : g.K * g.a_cs) * 4);
  p.b_bytes = (uint32_t)((B_KC ? g.N * g.b_rs : g.K * g.b_cs) * 4);
  p.c_bytes = (uint32_t)(g.M * g.ldc * 4);
  static bool attr_set = false;  // per instantiation
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_f32_split_kernel<A_KC, B_KC, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds) != hipSuccess)
    return fail(TM_ELAUNCH, "gemm_f32_split: cannot reserve %d bytes of LDS", kSplitLds);
  attr_set = true;
  const int64_t blocks = (int64_t)p.tiles_m * p.tiles_n;
  if (blocks > 0x7fffffff) return fail(TM_ESIZE, "gemm_f32_split: too many tiles");
  g_last_kernel = "gemm_f32_split_kernel";
  gemm_f32_split_kernel<A_KC, B_KC, EPI><<<(unsigned)blocks, 512, kSplitLds, s>>>(p);
  return check_launch("gemm_f32_split");
}

bool gemm_f32_split_supported(const GemmArgs &g) {
  return gemm_f32_supported(g) && g.N % 4 == 0 && g.ldc % 4 == 0 && (((uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.residual) & 15) == 0;
}

int gemm_f32_split(const GemmArgs &g, hipStream_t s) {
  if (g.c_mode == 1) return launch<false, false, 1>(g, s);
  if (g.c_mode == 2) return launch<false, false, 2>(g, s);
  return g.b_cs == 1 ? launch<true, true, 0>(g, s) : launch<true, false, 0>(g, s);
}

}  // namespace tmk
