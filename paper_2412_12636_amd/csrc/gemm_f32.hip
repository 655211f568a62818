// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation), the products of the fp32
// stage dtype.
//
// A step is 32 elements of the reduction axis.  Operand tiles go straight into LDS (buffer_load ... lds, 16 bytes per
// lane), several steps ahead:
//   * contiguous reduction axis: LDS tile [row][32], 16-byte chunks XOR-swizzled by row; a lane reads four reduction
//     elements of its row at once, 8j + 4hh .. +3 (hh: half of the wave), and they feed four MFMAs one by one;
//   * strided reduction axis: LDS tile [k][rows], the global layout; a lane reads element (8j + 4hh + i, row).
// Both kinds pair the reduction elements the same way, so any two layouts combine.
//
// Bound by the MFMA rate: 64 clocks for 32x32x2, a quarter of a wave's 64x64 tile per pair of reduction elements, for
// which LDS delivers 16 bytes per clock and unit and L2 eight.  What decides the time of a small product is therefore how
// evenly its tiles cover the SIMDs, and how much of the barrier and the LDS latency a second wave of the SIMD covers:
// blocks of 128x128 and 64x64, one wave a SIMD; of 64x64 with four waves a SIMD, and of 32x32 with one or two, that split
// every stage's reduction elements (their sums meet in LDS in wave order); and of 16x16, split four ways, on 16x16x4 MFMAs,
// where 32x32 tiles leave most units without one.  Which one: gemm_f32_form.h.  Larger products go to the bf16 instructions in
// three terms an element (gemm_f32_split.hip).
// With one wave a SIMD on every tile and none of 16x16 before: 1024 x 1024 over 1024 23.7 -> 21.9 us, over 3072 (strided
// weights) 64 -> 58; 256 x 256 over 1024 8.2 -> 4.5; 1500 x 768 over 768 25.1 -> 24.2 (weight gradient 29.9 -> 25.4).
// (The twelve products of a layer of hidden 1024, SwiGLU width 4096, 1024 tokens: 4.9 ms = 21 TFLOP/s on the 64x64
// plain-ALU tile kernel that this one replaces, 1.03 ms = 100 TFLOP/s here; its largest run at 113, the vendor BLAS reaches
// 150 on 8192^3.  The matrix cores are busy for 80 to 84 % of the cycles in which a unit has waves on 128x128 tiles, 69 % on
// 64x64.)
#include "act.h"
#include "gemm.h"
#include "gemm_f32_form.h"

namespace tmk {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int FK = 32;     // reduction elements of a step
constexpr int kPatch = 8;  // row-tiles of a patch
constexpr int kPairBlocks = 512;  // tiles of either gradient up to which the two share a launch: two a unit, what fits at once

struct F32GemmParams {
  int M, N, K;
  const float *A, *B;
  int64_t lda, ldb;  // the non-unit strides
  float *C;
  int64_t ldc;
  const float *bias, *residual;
  int tiles_m, tiles_n;
  uint32_t a_bytes, b_bytes, c_bytes;
  const float *u;  // EPI 4
  float *g;        // EPI 3
  int act;
};

// Loaders: NW waves fetch a step's tile of R rows.  MF: rows of an MFMA (32: 32x32x2, a lane reads elements 8j + 4hh .. +3;
// 16: 16x16x4, elements 16j + 4g .. +3, g: quarter of the wave).
//
// element (r, k) at base[r*ld + k]; LDS [R][32]
template <int R, int NW, int MF> struct F32KC {
  static constexpr int NLOAD = R * FK * 4 / 1024 / NW, BYTES = R * FK * 4;
  static __device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }
  uint32_t voff[NLOAD];
  int chunk[NLOAD], k_end;
  __device__ __forceinline__ void init(int64_t ld, int row0, int K, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int row = (i * NW + wave) * 8 + lane / 8;
      chunk[i] = ((lane % 8) ^ swz(row)) * 4;
      voff[i] = (uint32_t)(((int64_t)(row0 + row) * ld + chunk[i]) * 4);
    }
    k_end = K;
  }
  // chunks past the end of the reduction hold the next row's elements: their lanes read outside the tensor (zero)
  __device__ __forceinline__ void issue(rsrc_t rs, char *tile, int k0, int64_t, int wave) const {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(tile + (i * NW + wave) * 1024), 16,
                                               k0 + chunk[i] < k_end ? voff[i] : 0x80000000u, (uint32_t)k0 * 4u, 0, 0);
  }
  static __device__ __forceinline__ f32x4 frag(const char *tile, int r0, int j, int lane) {
    const int r = r0 + lane % MF;
    return *reinterpret_cast<const f32x4 *>(tile + r * FK * 4 + (((64 / MF * j + lane / MF) ^ swz(r)) << 4));
  }
};

// element (r, k) at base[k*ld + r]; LDS [32][R].  The two halves of a wave read k-rows that are four apart: XOR of one
// chunk bit with k bit 2 sends them to different 128-byte halves (R = 32 has only one).  R = 16: the four quarters of a wave
// read rows of 64 bytes that are four apart; row 4a + b of each 16 sits at 4b + a, so that they lie side by side.
template <int R, int NW, int MF> struct F32KS {
  static constexpr int CPR = R / 4, NLOAD = R * FK * 4 / 1024 / NW, BYTES = R * FK * 4;
  static __device__ __forceinline__ int swz(int kk) { return CPR >= 16 ? ((kk >> 2) & 1) << 3 : 0; }
  static __device__ __forceinline__ int slot(int kk) { return R == 16 ? (kk & 16) | ((kk & 3) << 2) | ((kk >> 2) & 3) : kk; }
  uint32_t voff[NLOAD];
  __device__ __forceinline__ void init(int64_t ld, int row0, int, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int idx = (i * NW + wave) * 64 + lane, kk = slot(idx / CPR), c = (idx % CPR) ^ swz(kk);
      voff[i] = (uint32_t)(((int64_t)kk * ld + row0 + c * 4) * 4);
    }
  }
  __device__ __forceinline__ void issue(rsrc_t rs, char *tile, int k0, int64_t ld, int wave) const {
    const uint32_t koff = (uint32_t)((int64_t)k0 * ld * 4);  // in the checked offset: rows past the end read as zero
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(tile + (i * NW + wave) * 1024), 16, voff[i] + koff, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 frag(const char *tile, int r0, int j, int lane) {
    const int r = r0 + lane % MF, g = lane / MF;
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kk = 256 / MF * j + 4 * g + i;
      x[i] = *reinterpret_cast<const float *>(tile + slot(kk) * R * 4 + (((r >> 2) ^ swz(4 * g)) << 4) + ((r & 3) << 2));
    }
    return x;
  }
};
template <int R, int NW, int MF, bool KC> struct F32Sel { typedef F32KC<R, NW, MF> type; };
template <int R, int NW, int MF> struct F32Sel<R, NW, MF, false> { typedef F32KS<R, NW, MF> type; };
template <int MF> struct F32Mma {
  static constexpr int NV = 16;
  typedef f32x16 acc_t;
  static __device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
};
template <> struct F32Mma<16> {
  static constexpr int NV = 4;
  typedef f32x4 acc_t;
  static __device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int v, int lane) { return 4 * (lane >> 4) + v; }
};

// WM, WN: wave tile (below 32: 16x16 MFMAs); KSPL: waves that split a stage's reduction elements; NS: LDS stages; SUB: steps
// of a stage, for tiles whose single step is shorter than the barrier and the LDS latency around it.  PATCH: the order of the
// walk, a form of its own (its arithmetic ahead of the first load cost the others 1 to 3 %, and weight gradients of four
// 64x64 tiles a unit 8 %: 4784 x 776 over 1324 94 -> 102 us)
template <int BM, int BN, int WM, int WN, int KSPL, int NS, int SUB> struct F32Cfg {
  static constexpr int MF = WM < 32 ? 16 : 32, NT = (BM / WM) * (BN / WN), NW = NT * KSPL;
  static constexpr int TM = WM / MF, TN = WN / MF, NV = F32Mma<MF>::NV;
  // a step of a small tile is fewer wave-wide loads than there are waves: groups of LW waves fetch alternate steps
  static constexpr int LW = NW * 1024 <= (BM < BN ? BM : BN) * FK * 4 ? NW : (BM < BN ? BM : BN) * FK * 4 / 1024, UG = NW / LW;
  static constexpr int STEP = (BM + BN) * FK * 4, STAGE = SUB * STEP, J = 4 * MF / 32;  // fragments of four elements a step
  static constexpr int WJ = KSPL < J ? KSPL : J, JW = J / WJ;  // split waves on the fragments of one step, and how many each takes
  static constexpr int SUMS = KSPL > 1 ? NW * NV * 256 : 0, LDS = NS * STAGE > SUMS ? NS * STAGE : SUMS;
  static_assert(KSPL == 1 || (TM == 1 && TN == 1 && NV % KSPL == 0), "split waves hold one tile each");
  static_assert(SUB % UG == 0 && SUB * J % KSPL == 0 && J % WJ == 0 && KSPL % WJ == 0, "steps divide among the waves");
};
// EPI 0: results with bias and residual.  1: added to C.  2: stored.  3: results with bias, and their GeLU to g.  4: results
// times the derivative of GeLU at u.
// One block's tile.  The thread's number and LDS are taken here, not handed in: the compiler then knows their ranges and folds the
// LDS addresses of strided operands into the reads (handed in, four reads of 4 bytes for every second step of a split 64x64 tile:
// input gradients 2.1 % slower, geometric mean over nine of 1000 to 8000 columns; 1024 x 1024 over 8192 140 -> 147 us).
template <int BM, int BN, int WM, int WN, int KSPL, int NS, int SUB, bool PATCH, bool A_KC, bool B_KC, int EPI>
__device__ __forceinline__ void f32_block(const F32GemmParams &p, const int lds_at, const unsigned block) {
  extern __shared__ __align__(1024) char all_lds[];
  char *const lds = all_lds + lds_at;
  typedef F32Cfg<BM, BN, WM, WN, KSPL, NS, SUB> C;
  typedef F32Mma<C::MF> MM;
  constexpr int MF = C::MF, TM = C::TM, TN = C::TN, NT = C::NT, LW = C::LW, UG = C::UG, NV = C::NV;
  typedef typename F32Sel<BM, LW, MF, A_KC>::type LA;
  typedef typename F32Sel<BN, LW, MF, B_KC>::type LB;
  constexpr int LOADS = SUB / UG * (LA::NLOAD + LB::NLOAD);
  int m0, n0;
  if constexpr (PATCH) {  // an XCD (ids round-robin over eight) owns a range of tiles, walked in patches
    asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.lda), "s"(p.ldb), "s"(p.K), "s"(p.a_bytes));  // fetched now, not behind the divisions
    const int nblk = p.tiles_m * p.tiles_n, xcd = (int)(block % 8), base = nblk / 8, rem = nblk % 8;
    const int lid = xcd * base + (xcd < rem ? xcd : rem) + (int)(block / 8);
    const int gi = lid / (kPatch * p.tiles_n), first = gi * kPatch, in_group = lid - first * p.tiles_n;
    const int rows = p.tiles_m - first < kPatch ? p.tiles_m - first : kPatch;
    m0 = (first + in_group % rows) * BM;
    n0 = (in_group / rows) * BN;
  } else {
    m0 = (int)(block % p.tiles_m) * BM;
    n0 = (int)(block / p.tiles_m) * BN;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % C::NW;
  // (zeros that the compiler can see: 5 % of the short products)
  const int ks = KSPL > 1 ? wave / NT : 0, wt = KSPL > 1 ? wave % NT : wave;
  const int lw = UG > 1 ? wave % LW : wave, lu = UG > 1 ? wave / LW : 0;
  const int wm = (wt / (BN / WN)) * WM, wn = (wt % (BN / WN)) * WN;
  LA la;
  LB lb;
  const rsrc_t ra = make_rsrc(p.A, p.a_bytes), rb = make_rsrc(p.B, p.b_bytes);
  la.init(p.lda, m0, p.K, lw, lane);
  lb.init(p.ldb, n0, p.K, lw, lane);
  typename MM::acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[i][j][v] = 0.f;
  const int nk = (p.K + SUB * FK - 1) / (SUB * FK);
  auto issue = [&](int stage) {  // steps past the end of the reduction read as zero
    char *st = lds + (stage % NS) * C::STAGE;
#pragma unroll
    for (int i = 0; i < SUB / UG; ++i) {
      const int u = i * UG + lu, k0 = (stage * SUB + u) * FK;
      la.issue(ra, st + u * C::STEP, k0, p.lda, lw);
      lb.issue(rb, st + u * C::STEP + LA::BYTES, k0, p.ldb, lw);
    }
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) issue(s);
  for (int kt = 0; kt < nk; ++kt) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * LOADS) : "memory");  // own loads of stage kt have landed
    __builtin_amdgcn_s_barrier();  // everyone's have; everyone has read stage kt - 1
    issue(kt + NS - 1);
#pragma unroll
    for (int i0 = 0; i0 < SUB * C::J / KSPL; ++i0) {
      const int j = i0 % C::JW * C::WJ + ks % C::WJ, u = i0 / C::JW * (KSPL / C::WJ) + ks / C::WJ;
      const char *As = lds + (kt % NS) * C::STAGE + u * C::STEP, *Bs = As + LA::BYTES;
      f32x4 a[TM], b[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t) a[t] = LA::frag(As, wm + t * MF, j, lane);
#pragma unroll
      for (int t = 0; t < TN; ++t) b[t] = LB::frag(Bs, wn + t * MF, j, lane);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = MM::mma(a[tm][i], b[tn][i], acc[tm][tn]);
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // the look-ahead loads, before LDS is reused or the block exits

  constexpr int VC = NV / KSPL;
  const int v_first = ks * VC;
  if constexpr (KSPL > 1) {  // a wave finishes VC registers of its tile, over all split waves in order
    __syncthreads();
    float *x = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[(wave * NV + v) * 64 + lane] = acc[0][0][v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < VC; ++e) {
      float s = x[(wt * NV + v_first + e) * 64 + lane];
#pragma unroll
      for (int w = 1; w < KSPL; ++w) s += x[((w * NT + wt) * NV + v_first + e) * 64 + lane];
      acc[0][0][e] = s;
    }
  }
  const rsrc_t rc = make_rsrc(p.C, p.c_bytes);
  const rsrc_t raux = make_rsrc(EPI == 3 ? p.g : EPI == 4 ? p.u : p.residual ? p.residual : p.C, p.c_bytes);
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    const int col = n0 + wn + tn * MF + lane % MF;
    const float bias = (EPI == 0 || EPI == 3) && p.bias && col < p.N ? p.bias[col] : 0.f;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      uint32_t off[VC];
      float old[VC];
#pragma unroll
      for (int e = 0; e < VC; ++e) {
        const int row = m0 + wm + tm * MF + MM::row(v_first + e, lane);
        off[e] = col < p.N && row < p.M ? (uint32_t)(((int64_t)row * p.ldc + col) * 4) : 0xfffffff0u;
        old[e] = 0.f;
      }
      if (EPI == 1 || EPI == 4 || (EPI == 0 && p.residual)) {
#pragma unroll
        for (int e = 0; e < VC; ++e)
          old[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(EPI == 1 ? rc : raux, off[e], 0, 0));
      }
#pragma unroll
      for (int e = 0; e < VC; ++e) {
        const float o = EPI == 4   ? acc[tm][tn][e] * gelu_grad_f(p.act, old[e])
                        : EPI == 0 ? (acc[tm][tn][e] + bias) + old[e]
                        : EPI == 3 ? acc[tm][tn][e] + bias
                                   : old[e] + acc[tm][tn][e];
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, o), rc, off[e], 0, 0);
        if (EPI == 3) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, gelu_f(p.act, o)), raux, off[e], 0, 0);
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int KSPL, int NS, int SUB, bool PATCH, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__((64 * F32Cfg<BM, BN, WM, WN, KSPL, NS, SUB>::NW)) void gemm_f32_kernel(const F32GemmParams p) {
  f32_block<BM, BN, WM, WN, KSPL, NS, SUB, PATCH, A_KC, B_KC, EPI>(p, 0, blockIdx.x);
}

// Input gradient and weight gradient of one linear map in one launch: blocks of DT x DT results of the first, then blocks of
// WT x WT of the second.  Both read the same output gradient and neither waits for the other; small ones, each a few
// microseconds of launch, first loads and epilogue around a few hundred cycles of MFMAs, cover each other: 16x16 tiles of both 6.7
// -> 3.7 us, 32x32 ones 9.3 -> 8.0.  Blocks of eight waves with 32x32 weight-gradient tiles split eight ways, whose 16x16 tiles of
// the input gradient come in pairs.  With GeLU and its derivative in the epilogues too, a step of one layer of hidden 256, FC of
// 1024: 33 tokens 88 -> 75 us, 512 127 -> 114, 1024 164 -> 155; the tiny preset's step 198 -> 178.
template <int DT, int WT, int WSPL> struct F32Pair {
  static constexpr int NW = WSPL, TWO = DT == 16 && WSPL == 8 ? 2 : 1, DSPL = DT == 16 ? 4 : WSPL, DSUB = TWO == 2 ? 2 : DT == 16 ? 4 : 2;
  typedef F32Cfg<DT, DT, DT, DT, DSPL, 4, DSUB> D;
  typedef F32Cfg<WT, WT, WT, WT, WSPL, 4, WT == 16 ? 4 : 2> W;
  static constexpr int LDS = TWO * D::LDS > W::LDS ? TWO * D::LDS : W::LDS;
  static_assert(D::NW * TWO == NW && W::NW == NW && 2 * LDS <= 160 * 1024, "blocks of one size, two to a unit");
};
template <int DT, int WT, int WSPL, int DEPI, int WEPI>
__global__ __launch_bounds__((64 * F32Pair<DT, WT, WSPL>::NW)) void gemm_f32_pair_kernel(const F32GemmParams d, const F32GemmParams w,
                                                                                         const int d_blocks) {
  typedef F32Pair<DT, WT, WSPL> P;
  if ((int)blockIdx.x < d_blocks) {
    // (a tile behind the last one, of an odd number, starts past the last column: it reads rows of the operands that are there,
    // the next reduction row's elements or zeros past the end, and stores nothing)
    const int sub = P::TWO == 2 ? (int)(threadIdx.x / 256) : 0;
    f32_block<DT, DT, DT, DT, P::DSPL, 4, P::DSUB, false, true, false, DEPI>(d, sub * P::D::LDS, blockIdx.x * P::TWO + sub);
  } else {
    f32_block<WT, WT, WT, WT, WSPL, 4, WT == 16 ? 4 : 2, false, false, false, WEPI>(w, 0, blockIdx.x - d_blocks);
  }
}

#define TM_F32_GEMM(W32, AKC, BKC, EPI)                                                                            \
  template __global__ void gemm_f32_kernel<128, 128, 64, 64, 1, 2, 1, false, AKC, BKC, EPI>(const F32GemmParams); \
  template __global__ void gemm_f32_kernel<64, 64, 32, 32, 1, 3, 1, false, AKC, BKC, EPI>(const F32GemmParams);   \
  template __global__ void gemm_f32_kernel<64, 64, 32, 32, 4, 3, 2, false, AKC, BKC, EPI>(const F32GemmParams);   \
  template __global__ void gemm_f32_kernel<32, 32, 32, 32, 4, 4, 2, false, AKC, BKC, EPI>(const F32GemmParams);   \
  template __global__ void gemm_f32_kernel<32, 32, 32, 32, W32, 4, 2, true, AKC, BKC, EPI>(const F32GemmParams);  \
  template __global__ void gemm_f32_kernel<16, 16, 16, 16, 4, 4, 4, false, AKC, BKC, EPI>(const F32GemmParams);
TM_F32_GEMM(4, true, true, 0)
TM_F32_GEMM(4, true, false, 0)
TM_F32_GEMM(8, false, false, 1)
TM_F32_GEMM(8, false, false, 2)
template __global__ void gemm_f32_kernel<32, 32, 32, 32, 4, 4, 2, false, true, true, 3>(const F32GemmParams);
template __global__ void gemm_f32_kernel<16, 16, 16, 16, 4, 4, 4, false, true, true, 3>(const F32GemmParams);
#define TM_F32_PAIR(DT, WT, WSPL)                                                                                  \
  template __global__ void gemm_f32_pair_kernel<DT, WT, WSPL, 0, 1>(const F32GemmParams, const F32GemmParams, int); \
  template __global__ void gemm_f32_pair_kernel<DT, WT, WSPL, 0, 2>(const F32GemmParams, const F32GemmParams, int); \
  template __global__ void gemm_f32_pair_kernel<DT, WT, WSPL, 4, 1>(const F32GemmParams, const F32GemmParams, int); \
  template __global__ void gemm_f32_pair_kernel<DT, WT, WSPL, 4, 2>(const F32GemmParams, const F32GemmParams, int);
TM_F32_PAIR(16, 16, 4)
TM_F32_PAIR(32, 16, 4)
TM_F32_PAIR(16, 32, 4)
TM_F32_PAIR(32, 32, 4)
TM_F32_PAIR(16, 32, 8)
TM_F32_PAIR(32, 32, 8)
template __global__ void gemm_f32_kernel<16, 16, 16, 16, 4, 4, 4, true, true, true, 0>(const F32GemmParams);
template __global__ void gemm_f32_kernel<16, 16, 16, 16, 4, 4, 4, true, true, false, 0>(const F32GemmParams);
template __global__ void gemm_f32_kernel<32, 32, 32, 32, 8, 4, 2, false, false, false, 1>(const F32GemmParams);
template __global__ void gemm_f32_kernel<32, 32, 32, 32, 8, 4, 2, false, false, false, 2>(const F32GemmParams);

// One of each operand's strides is 1, 16-byte chunks along it are aligned and whole, 32-bit offsets reach everything.
bool gemm_f32_supported(const GemmArgs &g) {
  auto operand_ok = [&](const void *ptr, int64_t rs, int64_t cs, int64_t rows) {
    if (((uintptr_t)ptr) & 15) return false;
    if (cs == 1) return rs % 4 == 0 && g.K % 4 == 0 && rows * rs * 4 < (1LL << 31);
    if (rs == 1) return cs % 4 == 0 && rows % 4 == 0 && g.K * cs * 4 < (1LL << 31) && (g.K + 2 * FK) * cs * 4 < (1LL << 32);
    return false;
  };
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.M > 0x3fffffff || g.N > 0x3fffffff || g.K > 0x3fffffff || g.c_mode > 2) return false;
  if (!operand_ok(g.A, g.a_rs, g.a_cs, g.M) || !operand_ok(g.B, g.b_rs, g.b_cs, g.N)) return false;
  if (g.M * g.ldc * 4 >= (1LL << 31)) return false;
  return g.c_mode ? (g.a_cs != 1 && g.b_cs != 1) : g.a_cs == 1;
}

static F32GemmParams make_params(const GemmArgs &g, int tile) {
  const bool a_kc = g.a_cs == 1, b_kc = g.b_cs == 1;
  F32GemmParams p;
  p.M = (int)g.M;
  p.N = (int)g.N;
  p.K = (int)g.K;
  p.A = (const float *)g.A;
  p.lda = a_kc ? g.a_rs : g.a_cs;
  p.B = (const float *)g.B;
  p.ldb = b_kc ? g.b_rs : g.b_cs;
  p.C = (float *)g.C;
  p.ldc = g.ldc;
  p.bias = (const float *)g.bias;
  p.residual = (const float *)g.residual;
  p.u = (const float *)g.act_u;
  p.g = (float *)g.act_g;
  p.act = g.act;
  p.tiles_m = (int)ceil_div(g.M, tile);
  p.tiles_n = (int)ceil_div(g.N, tile);
  p.a_bytes = (uint32_t)((a_kc ? g.M * g.a_rs : g.K * g.a_cs) * 4);
  p.b_bytes = (uint32_t)((b_kc ? g.N * g.b_rs : g.K * g.b_cs) * 4);
  p.c_bytes = (uint32_t)(g.M * g.ldc * 4);
  return p;
}

template <int BM, int BN, int WM, int WN, int KSPL, int NS, int SUB, bool PATCH, bool A_KC, bool B_KC, int EPI>
static int launch(const GemmArgs &g, hipStream_t s) {
  const F32GemmParams p = make_params(g, BM);
  typedef F32Cfg<BM, BN, WM, WN, KSPL, NS, SUB> C;
  constexpr int lds = C::LDS;
  static bool attr_set = false;  // per instantiation
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_f32_kernel<BM, BN, WM, WN, KSPL, NS, SUB, PATCH, A_KC, B_KC, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
    return fail(TM_ELAUNCH, "gemm_f32: cannot reserve %d bytes of LDS", lds);
  attr_set = true;
  const int64_t blocks = (int64_t)p.tiles_m * ceil_div(g.N, BN);
  if (blocks > 0x7fffffff) return fail(TM_ESIZE, "gemm_f32: too many tiles");
  g_last_kernel = "gemm_f32_kernel";
  gemm_f32_kernel<BM, BN, WM, WN, KSPL, NS, SUB, PATCH, A_KC, B_KC, EPI><<<(unsigned)blocks, 64 * C::NW, lds, s>>>(p);
  return check_launch("gemm_f32");
}

// the last stage of the 16x16 form reaches 4 FK rows past a strided operand's end: their offsets must not come round to its front
static bool reach16(const GemmArgs &g) {
  auto reaches = [&](int64_t cs) { return cs == 1 || (g.K + 4 * FK) * cs * 4 < (1LL << 32); };
  return reaches(g.a_cs) && reaches(g.b_cs);
}

template <bool A_KC, bool B_KC, int EPI> static int pick(const GemmArgs &g, hipStream_t s) {
  if (gemm_f32_split_supported(g) && f32_split(g.M, g.N, g.K, EPI != 0, reach16(g))) return gemm_f32_split(g, s);
  const F32Form f = f32_form(g.M, g.N, g.K, EPI != 0, reach16(g));
  if (f.tile == 128) return launch<128, 128, 64, 64, 1, 2, 1, false, A_KC, B_KC, EPI>(g, s);
  if (f.tile == 64 && f.split == 4) return launch<64, 64, 32, 32, 4, 3, 2, false, A_KC, B_KC, EPI>(g, s);
  if (f.tile == 64) return launch<64, 64, 32, 32, 1, 3, 1, false, A_KC, B_KC, EPI>(g, s);
  if (f.tile == 32 && f.patches) return launch<32, 32, 32, 32, EPI ? 8 : 4, 4, 2, true, A_KC, B_KC, EPI>(g, s);
  if constexpr (EPI != 0) {
    if (f.tile == 32 && f.split == 8) return launch<32, 32, 32, 32, 8, 4, 2, false, A_KC, B_KC, EPI>(g, s);
  } else {
    if (f.tile == 16 && f.patches) return launch<16, 16, 16, 16, 4, 4, 4, true, A_KC, B_KC, EPI>(g, s);
  }
  if (f.tile == 32) return launch<32, 32, 32, 32, 4, 4, 2, false, A_KC, B_KC, EPI>(g, s);
  return launch<16, 16, 16, 16, 4, 4, 4, false, A_KC, B_KC, EPI>(g, s);
}

// f32_form's choice where it is a small tile walked in plain order and no other kernel has the product
static bool small_form(const GemmArgs &g, bool wgrad, F32Form *f) {
  if (!gemm_f32_supported(g)) return false;
  *f = f32_form(g.M, g.N, g.K, wgrad, reach16(g));
  return f->tile <= 32 && !f->patches && !(gemm_f32_split_supported(g) && f32_split(g.M, g.N, g.K, wgrad, reach16(g)));
}

template <int DT, int WT, int WSPL, int DEPI, int WEPI> static int launch_pair(const GemmArgs &d, const GemmArgs &w, hipStream_t s) {
  typedef F32Pair<DT, WT, WSPL> P;
  const F32GemmParams pd = make_params(d, DT), pw = make_params(w, WT);
  static bool attr_set = false;  // per instantiation
  if (!attr_set && hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_f32_pair_kernel<DT, WT, WSPL, DEPI, WEPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, P::LDS) != hipSuccess)
    return fail(TM_ELAUNCH, "gemm_f32_pair: cannot reserve %d bytes of LDS", P::LDS);
  attr_set = true;
  const int d_blocks = (int)ceil_div((int64_t)pd.tiles_m * pd.tiles_n, P::TWO);
  g_last_kernel = "gemm_f32_pair_kernel";
  gemm_f32_pair_kernel<DT, WT, WSPL, DEPI, WEPI><<<(unsigned)(d_blocks + pw.tiles_m * pw.tiles_n), 64 * P::NW, P::LDS, s>>>(pd, pw, d_blocks);
  return check_launch("gemm_f32_pair");
}
template <int DT, int WT, int WSPL> static int pick_pair(const GemmArgs &d, const GemmArgs &w, hipStream_t s) {
  if (d.act_u) return w.c_mode == 1 ? launch_pair<DT, WT, WSPL, 4, 1>(d, w, s) : launch_pair<DT, WT, WSPL, 4, 2>(d, w, s);
  return w.c_mode == 1 ? launch_pair<DT, WT, WSPL, 0, 1>(d, w, s) : launch_pair<DT, WT, WSPL, 0, 2>(d, w, s);
}
bool gemm_f32_pair(const GemmArgs &d, const GemmArgs &w, hipStream_t s, int *status) {
  F32Form fd, fw;
  if (d.c_mode != 0 || d.b_cs == 1 || (w.c_mode != 1 && w.c_mode != 2) || !small_form(d, false, &fd) || !small_form(w, true, &fw)) return false;
  if (ceil_div(d.M, fd.tile) * ceil_div(d.N, fd.tile) > kPairBlocks || ceil_div(w.M, fw.tile) * ceil_div(w.N, fw.tile) > kPairBlocks) return false;
  if (!status) return true;
  if (fw.tile == 16) *status = fd.tile == 16 ? pick_pair<16, 16, 4>(d, w, s) : pick_pair<32, 16, 4>(d, w, s);
  else if (fw.split == 4) *status = fd.tile == 16 ? pick_pair<16, 32, 4>(d, w, s) : pick_pair<32, 32, 4>(d, w, s);
  else *status = fd.tile == 16 ? pick_pair<16, 32, 8>(d, w, s) : pick_pair<32, 32, 8>(d, w, s);
  return true;
}
bool gemm_f32_act(const GemmArgs &g, hipStream_t s, int *status) {
  F32Form f;
  if (g.c_mode != 0 || g.b_cs != 1 || g.residual || !small_form(g, false, &f)) return false;
  if (!status) return true;
  *status = f.tile == 16 ? launch<16, 16, 16, 16, 4, 4, 4, false, true, true, 3>(g, s) : launch<32, 32, 32, 32, 4, 4, 2, false, true, true, 3>(g, s);
  return true;
}

int gemm_f32(const GemmArgs &g, hipStream_t s) {
  if (g.c_mode == 1) return pick<false, false, 1>(g, s);
  if (g.c_mode == 2) return pick<false, false, 2>(g, s);
  return g.b_cs == 1 ? pick<true, true, 0>(g, s) : pick<true, false, 0>(g, s);
}

}  // namespace tmk
