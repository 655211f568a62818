// bf16 products of few output tiles: 32x32 results a block, the reduction split among its waves.
//
// A 64x64 tile walks its whole reduction in steps of 64 elements, about 0.17 us each however few of the units have a tile: 256 x
// 512 over 2048 are 32 tiles and 10.6 us.  Here a tile is a quarter of that, and every wave takes every NW-th chunk of 64
// elements through LDS of its own, so that no barrier stands in the main loop and what is left of the walk is its first loads'
// way from HBM or L2.  Bound by that latency, the launch and the meeting of the waves' sums (in wave order, in LDS).
//
// Loads go straight to LDS, NS chunks ahead, and are out of the compiler's sight (load_to_lds): a wave waits for its oldest
// chunk by count.  Chunks behind the end of the reduction are fetched too, from outside the tensors (zeros), which keeps
// that count the same for all of them.
#include <type_traits>

#include "gemm_mfma_impl.h"

namespace tmk {

constexpr int kChunkLoads = 8;  // wave-wide loads of a chunk, four of each operand

// element (r, k) at base[r*ld + k]; LDS [32][64], as DirectKC
struct SmallKC {
  typedef DirectKC<32, 64, 1, false> L;
  uint32_t voff[4];
  int k_lane;
  __device__ __forceinline__ void init(int64_t ld, int row0, int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 8 + lane / 8, c = (lane % 8) ^ L::swz(row);
      voff[i] = (uint32_t)(((int64_t)(row0 + row) * ld + c * 8) * 2);
      if (i == 0) k_lane = c * 8;  // of load i: this with chunk bits ^ i
    }
  }
  __device__ __forceinline__ void issue(rsrc_t rs, const char *tile, int k0, int K, int64_t) const {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      load_to_lds(rs, tile + i * 1024, k0 + (k_lane ^ (i * 8)) < K ? voff[i] : 0x80000000u, (uint32_t)k0 * 2u);
  }
  static __device__ __forceinline__ bf16x8 frag(const char *tile, int ks, int lane) { return L::frag(tile, 0, ks, lane); }
};
// element (r, k) at base[k*ld + r]; LDS [64][32]: the four k-rows of 64 bytes that half a wave's transposing read touches are
// the 64 banks in order
struct SmallKS {
  uint32_t voff[4];
  int k_lane;
  __device__ __forceinline__ void init(int64_t ld, int row0, int lane) {
    k_lane = lane / 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) voff[i] = (uint32_t)(((int64_t)(i * 16 + k_lane) * ld + row0 + lane % 4 * 8) * 2);
  }
  __device__ __forceinline__ void issue(rsrc_t rs, const char *tile, int k0, int K, int64_t ld) const {
    const uint32_t koff = (uint32_t)((int64_t)k0 * ld * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      load_to_lds(rs, tile + i * 1024, k0 + i * 16 + k_lane < K ? voff[i] + koff : 0x80000000u, 0);
  }
  static __device__ __forceinline__ bf16x8 frag(const char *tile, int ks, int lane) {
    const int g = lane >> 4, s = lane & 15;
    const char *a = tile + (16 * ks + 8 * (g >> 1) + (s >> 2)) * 64 + (16 * (g & 1) + 4 * (s & 3)) * 2;
    union { s16x4 h[2]; bf16x8 v; } x;
#pragma unroll
    for (int t = 0; t < 2; ++t)
      x.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(a + 4 * t * 64));
    return x.v;
  }
};

struct SmallCfg {
  static constexpr int NW = 4, NS = 2;  // waves; chunks of a wave in flight
  static constexpr int CHUNK = 2 * 32 * 64 * 2, PITCH = 65;  // floats: a register's row in the exchange, off the banks' round
  static constexpr int SUMS = NW * 16 * PITCH * 4, LDS = NW * NS * CHUNK;
  static_assert(LDS >= SUMS, "the sums meet where the chunks were");
};

template <bool B_KC>
__global__ __launch_bounds__(64 * SmallCfg::NW) void gemm_small_kernel(const MfmaGemmParams p) {
  typedef SmallCfg C;
  typedef SmallKC LA;
  constexpr int NW = C::NW, NS = C::NS;
  typedef std::conditional_t<B_KC, SmallKC, SmallKS> LB;
  extern __shared__ __align__(1024) char lds[];
  int m0, n0;
  tile_of_block(p, 32, 32, m0, n0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  LA la;
  LB lb;
  const rsrc_t ra = make_rsrc(p.A, p.a_bytes), rb = make_rsrc(p.B, p.b_bytes);
  la.init(p.lda, m0, lane);
  lb.init(p.ldb, n0, lane);
  char *const mine = lds + wave * NS * C::CHUNK;
  auto issue = [&](int c, const char *slot) {  // the wave's c-th chunk
    const int k0 = (c * NW + wave) * 64;
    la.issue(ra, slot, k0, p.K, p.lda);
    lb.issue(rb, slot + C::CHUNK / 2, k0, p.K, p.ldb);
  };
#pragma unroll
  for (int c = 0; c < NS; ++c) issue(c, mine + c * C::CHUNK);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int nk = (p.K + 63) / 64, chunks = (nk - wave + NW - 1) / NW;
  char *slot = mine;
  for (int c = 0; c < chunks; ++c) {
    wait_vmcnt<(NS - 1) * kChunkLoads>();  // loads land in order
    bf16x8 a[4], b[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      a[ks] = LA::frag(slot, ks, lane);
      b[ks] = LB::frag(slot + C::CHUNK / 2, ks, lane);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the chunk is in registers, its place is free
    asm volatile("" ::: "memory");
    issue(c + NS, slot);
    slot = slot == mine + (NS - 1) * C::CHUNK ? mine : slot + C::CHUNK;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b[ks], acc, 0, 0, 0);
  }
  wait_vmcnt<0>();  // what was fetched ahead, before the chunks' places are reused
  __syncthreads();
  float *x = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int v = 0; v < 16; ++v) x[(wave * 16 + v) * C::PITCH + lane] = acc[v];
  __syncthreads();
  // two neighbouring results a thread: register 4 (row / 8) + row % 4, lane 32 (row / 4 % 2) + column
  const rsrc_t rc = make_rsrc(p.C, p.c_bytes);
#pragma unroll
  for (int i = 0; i < 512 / (64 * NW); ++i) {
    const int t = i * 64 * NW + (int)threadIdx.x, row = t / 16, col = t % 16 * 2;
    const float *at = x + (4 * (row >> 3) + (row & 3)) * C::PITCH + 32 * ((row >> 2) & 1) + col;
    float r[2] = {at[0], at[1]};
#pragma unroll
    for (int w = 1; w < NW; ++w) r[0] += at[w * 16 * C::PITCH], r[1] += at[w * 16 * C::PITCH + 1];
    const int gm = m0 + row, gn = n0 + col;  // N is a multiple of 8
    const bool ok = gm < p.M && gn < p.N;
    const uint32_t off = ok ? (uint32_t)(((int64_t)gm * p.ldc + gn) * 2) : 0x80000000u;
    auto add = [&](uint32_t two) {
      r[0] += __builtin_bit_cast(float, two << 16);
      r[1] += __builtin_bit_cast(float, two & 0xffff0000u);
    };
    if (p.bias && ok) add(*reinterpret_cast<const uint32_t *>(p.bias + gn));
    if (p.residual) add(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(p.residual, p.c_bytes), off, 0, 0));
    const bf16 o[2] = {(bf16)r[0], (bf16)r[1]};
    uint32_t two;
    __builtin_memcpy(&two, o, 4);
    __builtin_amdgcn_raw_buffer_store_b32(two, rc, off, 0, 0);
  }
}

template <bool B_KC> static int launch_small(const GemmArgs &g, hipStream_t s) {
  MfmaGemmParams p = {};
  p.M = (int)g.M;
  p.N = (int)g.N;
  p.K = (int)g.K;
  p.A = (const bf16 *)g.A;
  p.lda = g.a_rs;
  p.B = (const bf16 *)g.B;
  p.ldb = B_KC ? g.b_rs : g.b_cs;
  p.C = g.C;
  p.ldc = g.ldc;
  p.bias = (const bf16 *)g.bias;
  p.residual = (const bf16 *)g.residual;
  p.tiles_m = (int)ceil_div(g.M, 32);
  p.tiles_n = (int)ceil_div(g.N, 32);
  p.a_bytes = (uint32_t)(g.M * g.a_rs * 2);
  p.b_bytes = (uint32_t)((B_KC ? g.N * g.b_rs : g.K * g.b_cs) * 2);
  p.c_bytes = (uint32_t)(g.M * g.ldc * 2);
  static_assert(SmallCfg::LDS <= 64 * 1024, "no LDS attribute needed, two blocks on a unit");
  g_last_kernel = "gemm_small_kernel";
  gemm_small_kernel<B_KC><<<(unsigned)(p.tiles_m * p.tiles_n), 64 * SmallCfg::NW, SmallCfg::LDS, s>>>(p);
  return check_launch("gemm_small");
}

// bf16 results over 1024 elements and more, with a tile on every unit at most, or two where both operands lie along the
// reduction.  Input gradients with scratch are asked about only where gemm_mfma() does not split their reduction (split_pays in
// gemm_mfma.hip).  Against the unsplit tiles chosen before, 1900 random products of each kind (8 to 4096 rows, 64 to 8192 columns, 64 to 12288
// elements), forward / input gradient, geometric means over up to 256 tiles: 0.60 / 0.67 of the time to 2048 elements, 0.51 / 0.61 to
// 4096, 0.46 / 0.60 beyond; 257 to 384 tiles 0.85 / 1.03, to 512 0.90 / 1.09 (one in sixty forward ones 4 to 7 % slower), to 560 1.20 /
// 1.45.  256 x 512 over 2048 10.6 -> 4.9 us.  With eight waves, or three or four chunks in flight, 2 to 10 % slower; 64x64 tiles
// split the same way as fast as the unsplit ones at best.  Shorter reductions (0.92 to 0.72) keep the tiles whose sums
// all configurations share bit for bit, and so do weight gradients, which have them with the update in the epilogue.
bool gemm_mfma_small_pays(const GemmArgs &g) {
  if (g.c_mode != 0 || g.N % 8 != 0 || g.K < 1024) return false;
  const int64_t tiles = ceil_div(g.M, 32) * ceil_div(g.N, 32);
  return tiles <= (g.b_cs == 1 ? 512 : 256);
}
int gemm_mfma_small(const GemmArgs &g, hipStream_t s) { return g.b_cs == 1 ? launch_small<true>(g, s) : launch_small<false>(g, s); }

}  // namespace tmk
