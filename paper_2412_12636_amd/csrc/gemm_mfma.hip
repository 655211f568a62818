// bf16 GEMM through the matrix cores: layout dispatch and choice of the tile configuration.  The kernels
// live in gemm_mfma_impl.h and are instantiated in one translation unit per operand layout.
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "gemm.h"

namespace tmk {

int gemm_mfma_nt(const GemmArgs &g, int config, hipStream_t s);  // y = x W^T       (both reduction axes contiguous)
int gemm_mfma_nn(const GemmArgs &g, int config, hipStream_t s);  // dx = dy W       (W read along its strided axis)
int gemm_mfma_tn(const GemmArgs &g, int config, hipStream_t s);  // dW (+)= dy^T x  (both strided, fp32 result)
int gemm_mfma_nn_partial(const GemmArgs &g, bool large, hipStream_t s);  // dx = dy W in k_splits fp32 parts
// bf16 results of few tiles, the reduction split among a block's waves (gemm_mfma_small.hip)
bool gemm_mfma_small_pays(const GemmArgs &g);
int gemm_mfma_small(const GemmArgs &g, hipStream_t s);

bool gemm_mfma_supported(const GemmArgs &g) {
  auto operand_ok = [&](const void *ptr, int64_t rs, int64_t cs, int64_t rows) {
    if (((uintptr_t)ptr) & 15) return false;
    if (cs == 1) return rs % 8 == 0 && g.K % 8 == 0;
    // (a ragged last step's rows past the end must not wrap around the 32-bit offset)
    if (rs == 1) return cs % 8 == 0 && rows % 8 == 0 && (g.K + 64) * cs * 2 < (1LL << 32);
    return false;
  };
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  if (g.M > 0x7fffffff || g.N > 0x7fffffff || g.K > 0x7fffffff) return false;
  if (!operand_ok(g.A, g.a_rs, g.a_cs, g.M) || !operand_ok(g.B, g.b_rs, g.b_cs, g.N)) return false;
  const bool akc = g.a_cs == 1, bkc = g.b_cs == 1;
  const int64_t a_bytes = (akc ? g.M * g.a_rs : g.K * g.a_cs) * 2, b_bytes = (bkc ? g.N * g.b_rs : g.K * g.b_cs) * 2;
  const int64_t c_bytes = g.M * g.ldc * (g.c_mode ? 4 : 2);
  if (a_bytes >= (1LL << 31) || b_bytes >= (1LL << 31) || c_bytes >= (1LL << 31)) return false;  // 32-bit offsets
  // the rows that the last tile has past the result are written outside it, not round 2^32 to its front
  if ((g.M + 256) * g.ldc * (g.c_mode ? 4 : 2) >= (1LL << 32)) return false;
  if (g.ldc % 8 || (((uintptr_t)g.C) & 15)) return false;
  return g.c_mode ? (!akc && !bkc) : akc;
}

// ---- tile configurations -------------------------------------------------------------------------
// Same order as TM_GEMM_CONFIGS in gemm_mfma_impl.h.  occ: blocks a compute unit holds at once (LDS: the stages of
// (BM+BN) x 128 bytes out of 160 KB).  Per operand layout (0: both reduction axes contiguous, 1: B strided, 2: both
// strided) what a product costs in microseconds: start, and per pass of blocks over the chip epi + steps of 64
// reduction elements at
//   one block on each unit:  alone + fill * (share of the units that have one: the others' power and bandwidth are free)
//   two blocks on a unit:    pair
// Fitted (relative least squares, 5 to 15 % rms) to every configuration's time on 146 products of 64 to 16384 rows,
// widths and reduction lengths from 128 to 20480, with weights that rotate through 400 MB.  The pick is 1 to 2.5 % slower
// than the fastest configuration on them (geometric mean); a model of relative speeds that took two blocks a unit for
// granted and knew no fixed cost was 50 to 61 % slower, most of it on products whose large tiles leave units idle.
struct LayoutCost {
  double start, alone, fill, pair, epi;
};
struct TileConfig {
  int bm, bn, wgm, wgn, occ;
  LayoutCost cost[3];
};
static const TileConfig kConfigs[] = {
    // the pipelined kernel
    {128, 192, 2, 2, 2,
     {{1.65, 0.608, 0.236, 1.334, 4.00}, {0.00, 0.835, 0.387, 1.320, 5.17}, {0.00, 0.714, 0.542, 1.364, 4.47}}},
    {128, 128, 2, 2, 2,
     {{0.00, 0.514, 0.216, 0.936, 4.08}, {0.01, 0.729, 0.273, 1.075, 3.85}, {0.00, 0.626, 0.346, 1.059, 3.87}}},
    {192, 128, 2, 2, 2,
     {{0.99, 0.572, 0.303, 1.325, 4.03}, {0.00, 0.817, 0.399, 1.295, 4.42}, {0.00, 0.752, 0.478, 1.378, 4.44}}},
    {256, 192, 4, 2, 1,
     {{0.00, 0.833, 0.519, 0.000, 6.06}, {0.00, 1.053, 0.499, 0.000, 5.39}, {0.00, 0.945, 0.645, 0.000, 5.16}}},
    {192, 256, 2, 4, 1,
     {{0.23, 0.831, 0.521, 0.000, 5.55}, {0.00, 1.049, 0.463, 0.000, 5.01}, {0.00, 1.033, 0.617, 0.000, 5.11}}},
    {256, 256, 2, 4, 1,
     {{0.00, 1.006, 0.647, 0.000, 6.50}, {0.00, 1.326, 0.551, 0.000, 5.54}, {0.00, 1.302, 0.727, 0.000, 5.69}}},
    {256, 256, 4, 2, 1,
     {{0.00, 1.015, 0.643, 0.000, 6.61}, {0.00, 1.288, 0.581, 0.000, 5.85}, {0.00, 1.183, 0.759, 0.000, 5.52}}},
    {256, 128, 4, 2, 1,
     {{1.35, 0.640, 0.387, 0.000, 3.55}, {0.67, 0.880, 0.372, 0.000, 3.61}, {0.00, 0.827, 0.410, 0.000, 4.29}}},
    {256, 192, 2, 2, 1,
     {{0.80, 0.928, 0.381, 0.000, 7.42}, {0.18, 1.330, 0.374, 0.000, 7.03}, {0.00, 1.159, 0.544, 0.000, 5.79}}},
    // the alternating kernel (gemm_alt_kernel)
    {256, 256, 2, 4, 1,
     {{0.00, 1.267, 0.542, 0.000, 6.75}, {0.00, 1.277, 0.420, 0.000, 6.34}, {0.00, 1.240, 0.540, 0.000, 6.74}}},
    {256, 256, 4, 2, 1,
     {{0.00, 1.269, 0.530, 0.000, 6.90}, {0.00, 1.276, 0.467, 0.000, 6.65}, {0.00, 1.196, 0.601, 0.000, 6.88}}},
    // the pipelined kernel with three LDS stages
    {256, 128, 4, 2, 1,
     {{0.49, 0.598, 0.301, 0.000, 4.77}, {0.67, 0.897, 0.350, 0.000, 3.78}, {0.00, 0.846, 0.379, 0.000, 4.59}}},
    {128, 256, 2, 4, 1,
     {{0.57, 0.576, 0.327, 0.000, 4.77}, {0.82, 0.930, 0.337, 0.000, 3.73}, {0.00, 0.830, 0.396, 0.000, 4.56}}},
    // the kernel with loader waves (gemm_ldw_kernel)
    {256, 192, 4, 2, 1,
     {{0.00, 0.740, 0.521, 0.000, 6.15}, {0.00, 0.769, 0.423, 0.000, 6.03}, {0.00, 0.683, 0.511, 0.000, 6.07}}},
    {128, 192, 2, 2, 2,
     {{0.00, 0.578, 0.292, 1.860, 5.20}, {0.00, 0.592, 0.264, 1.706, 5.04}, {0.00, 0.422, 0.447, 1.575, 4.81}}},
    {256, 192, 4, 2, 1,
     {{0.00, 0.752, 0.494, 0.000, 6.39}, {0.00, 0.769, 0.416, 0.000, 6.32}, {0.00, 0.686, 0.513, 0.000, 6.41}}},
    // ... on small tiles with more stages
    {64, 64, 2, 2, 2,
     {{2.49, 0.168, 0.030, 0.419, 1.91}, {2.67, 0.183, 0.036, 0.427, 1.41}, {2.38, 0.139, 0.076, 0.381, 1.51}}},
    {128, 64, 2, 2, 2,
     {{2.15, 0.246, 0.119, 0.680, 2.39}, {2.61, 0.283, 0.075, 0.708, 1.75}, {1.90, 0.280, 0.099, 0.654, 2.40}}},
    {64, 128, 2, 2, 2,
     {{1.91, 0.259, 0.106, 0.654, 2.71}, {2.41, 0.273, 0.080, 0.681, 2.17}, {1.90, 0.260, 0.090, 0.644, 2.38}}},
    {128, 128, 2, 2, 1,
     {{1.62, 0.299, 0.209, 0.000, 3.64}, {1.52, 0.320, 0.192, 0.000, 3.62}, {1.27, 0.286, 0.192, 0.000, 3.46}}},
};
constexpr int kNumConfigs = sizeof(kConfigs) / sizeof(kConfigs[0]);
constexpr int kDeep64x128Config = 18;  // index in kConfigs

static int layout_of(const GemmArgs &g) { return g.c_mode ? 2 : (g.b_cs == 1 ? 0 : 1); }

static double config_us(const GemmArgs &g, int c, int layout) {
  const TileConfig &t = kConfigs[c];
  const LayoutCost &k = t.cost[layout];
  const int64_t nb = ceil_div(g.M, t.bm) * ceil_div(g.N, t.bn);
  const double steps = (double)ceil_div(g.K, (int64_t)64);
  if (t.occ == 1) {
    const double passes = (double)ceil_div(nb, (int64_t)256);
    return k.start + passes * (k.epi + steps * (k.alone + k.fill * (double)nb / (256.0 * passes)));
  }
  const int64_t rest = nb % 512;
  const double pairs = (double)(nb / 512 + (rest > 256)), alone = rest > 0 && rest <= 256 ? 1.0 : 0.0;
  return k.start + (pairs + alone) * k.epi + steps * (pairs * k.pair + alone * (k.alone + k.fill * (double)rest / 256.0));
}
static bool config_takes(const GemmArgs &g, int c, int layout) {
  return g.K % 64 == 0 || layout == 2 || c == 1 || gemm_config_takes_ragged_k(c);
}
// A weight gradient whose rows do not start on 128-byte lines reads and writes two partial lines for every 32 results, through
// different blocks where a tile ends: with few tokens that, and not the main loop, is its time, and small tiles, whose
// epilogues overlap other blocks' main loops, lose least.  Time = scale x the model's + per million results, for results that
// are added to and that are overwritten, fitted to 393 and 199 such matrices.  On matrices left out of the fit the pick is
// 18 % and 9 % faster than the model's alone (the fastest configuration: 19 % and 14 %) and slower by more than 3 % on 10 and 8
// of them.  The range: below 2^23 results one matrix in six lost 3 to 28 %, and from some 1000 and 480 tokens on the model alone
// is as good.  40 tokens on 5128 x 3080 added to 50 -> 38 us, 300 on 8200 x 3080 104 -> 76 (overwritten 60 -> 50), 1000 on
// 5128 x 3080 91 -> 73.
struct OffLineCost {
  int config;
  double scale[2], per_million[2];  // added to, overwritten
};
static const OffLineCost kOffLine[] = {{13, {1.03, 0.83}, {2.40, 1.05}}, {14, {0.86, 0.81}, {2.39, 1.05}}, {17, {0.82, 0.72}, {1.72, 0.79}},
                                       {18, {0.77, 0.76}, {2.09, 0.80}}, {19, {0.87, 0.94}, {1.95, 0.54}}};
static int off_line_config(const GemmArgs &g) {  // -1: not such a product
  if ((g.c_mode != 1 && g.c_mode != 2) || (g.ldc % 32 == 0 && (((uintptr_t)g.C) & 127) == 0) || g.M * g.N < (1LL << 23)) return -1;
  const bool adds = g.c_mode == 1;
  if (adds ? g.K > 1024 : g.K <= 32 || g.K > 480) return -1;
  double best = 1e300;
  int pick = -1;
  for (const OffLineCost &o : kOffLine) {
    const double us = o.scale[!adds] * config_us(g, o.config, 2) + o.per_million[!adds] * ((double)g.M * g.N / 1e6);
    if (us < best) best = us, pick = o.config;
  }
  return pick;
}
static int heuristic_config(const GemmArgs &g) {
  double best = 1e300;
  int pick = 0;
  const int layout = layout_of(g);
  // An overwritten weight gradient of one reduction step and 32 M parameters or more is nothing but its fp32 results
  // leaving for HBM, which the model, fitted to products of two steps and more, does not know.  Small tiles spread the stores
  // most evenly; 48 tokens, model's tiles / 64 x 128: 16384 x 4096 65 / 54 us, 8192 x 8192 59 / 49, 12288 x 6144 62 / 54, 20480 x
  // 5120 85 / 75, 8192 x 16384 119 / 99.  (Added to, the same matrices have no best tiles: each loses 5 to 15 % on some.)
  if (g.c_mode == 2 && g.K <= 64 && g.M * g.N >= (1LL << 25)) return kDeep64x128Config;
  if (const int c = off_line_config(g); c >= 0) return c;
  for (int c = 0; c < kNumConfigs; ++c) {
    if (!config_takes(g, c, layout)) continue;
    const double us = config_us(g, c, layout);
    if (us < 0.99 * best) best = us, pick = c;  // near ties (the forms with four and with two loaders) go to the first
  }
  return pick;
}

// TM_GEMM_TILE=<BM>x<BN>x<WGM>x<WGN> in the environment forces one configuration (tuning aid).
static int g_override_config = -1;  // tm_gemm_force_config
static int forced_config() {
  if (g_override_config >= 0) return g_override_config;
  static int forced = -2;
  if (forced == -2) {
    forced = -1;
    if (const char *e = getenv("TM_GEMM_TILE")) {
      int a = 0, b = 0, c = 0, d = 0;
      if (sscanf(e, "%dx%dx%dx%d", &a, &b, &c, &d) == 4)
        for (int i = 0; i < kNumConfigs; ++i)
          if (kConfigs[i].bm == a && kConfigs[i].bn == b && kConfigs[i].wgm == c && kConfigs[i].wgn == d) forced = i;
    }
  }
  return forced;
}

int gemm_mfma_config_count() { return kNumConfigs; }
int gemm_mfma_force_config(int index) {
  if (index < -1 || index >= kNumConfigs) return fail(TM_EINVAL, "gemm_force_config: no configuration %d", index);
  g_override_config = index;
  return TM_OK;
}

// Configurations found by gemm_mfma_tune(), keyed by (layout, M, N, K).  A weight-gradient product that also applies
// the update (c_mode 3) has layout key 3: its choice weighs the stream of optimizer state against the main loop.
typedef std::tuple<int, int64_t, int64_t, int64_t> TuneKey;
static std::map<TuneKey, int> g_tuned;
static std::mutex g_tuned_mutex;
constexpr int kFusedLayoutKey = 3;

// Time of a fused-update product from the main loop's: many small blocks overlap one another's main loops and state
// streams (26 bytes per parameter, priced at 5 TB/s), large ones pull fewer operand bytes.  Fitted to 32 matrices of
// 768 x 768 to 12288 x 6144 parameters and 300 to 8192 tokens, on which it picks within 1 % of the fastest of nine
// configurations on average; two 128x192 or 128x128 blocks a unit for all of them were 30 % slower (1024 x 1024, 4000
// tokens: 69 -> 22 us on 64x64 tiles; 2048 x 4096, 2048 tokens: 83 -> 73).
struct FusedCost {
  int config;
  double main, stream, start;
};
static const FusedCost kFused[] = {{13, 0.70, 0.68, 24.8}, {14, 0.90, 0.49, 19.8}, {16, 0.99, 0.37, 3.0}, {19, 0.98, 0.69, 9.3}};
// main_us[c]: the plain product's measured time per configuration, or NULL for the model's
static int fused_config(const GemmArgs &g, const float *main_us) {
  double best = 1e300;
  int pick = kFused[0].config;
  const double stream_us = (double)g.M * g.N * 26 / 5e6;
  for (const FusedCost &f : kFused) {
    const double us = f.main * (main_us ? main_us[f.config] : config_us(g, f.config, 2)) + f.stream * stream_us + f.start;
    if (us < best) best = us, pick = f.config;
  }
  return pick;
}

// A fused-update product whose 256x192 tiles fill the chip at least twice and whose main loop is short enough for
// the update to matter (up to 4096 tokens) runs on the kernel with loader waves, one block per compute unit, with
// start offsets between the units (gemm_mfma_impl.h, stagger_by_unit): 0.53 -> 0.42 ms for the FC-sized matrices of
// the 175B shard.  TM_GEMM_FUSED_LARGE=0 switches this off, TM_GEMM_FUSED_LARGE_MAXT moves the token limit.
constexpr int kLdwLargeConfig = 13;
static bool fused_on_large_tiles(const GemmArgs &g) {
  static int on = -1;
  static int64_t max_t = 4096;
  if (on < 0) {
    const char *e = getenv("TM_GEMM_FUSED_LARGE");
    on = e ? atoi(e) != 0 : 1;
    if (const char *t = getenv("TM_GEMM_FUSED_LARGE_MAXT")) max_t = atoll(t);
  }
  const TileConfig &t = kConfigs[kLdwLargeConfig];
  return on && g.K <= max_t && ceil_div(g.M, t.bm) * ceil_div(g.N, t.bn) >= 512;
}

// The update in the epilogue streams a matrix's state row by row in segments of 32 parameters: whole 128-byte lines only
// where rows start on one.  Rows that do not make two partial lines of every segment, read and written by different blocks:
// a backward pass with updates, fused / flat, 7480 wide 1987 / 929 us at 82 tokens and 2330 / 1687 at 2048, 4104 wide 591 / 427
// and 1006 / 877, 1032 wide 239 / 172 and 411 / 355.
// A token count that is no multiple of 64 stores its gradients in every gradient mode, so that the epilogue saves only their
// reading back.  That pays on the large staggered form from some 700 tokens on (12288 wide, fused / flat: 82 tokens 1606 /
// 1462 us, 500 1914 / 1901, 1000 2299 / 2342, 2000 3191 / 3335; 8192 wide: 500 1306 / 1245, 1000 1596 / 1609), on small tiles
// nowhere (1024 wide: 82 tokens 236 / 216, 1000 333 / 330, 4000 762 / 747; 4096 wide: 82 tokens 469 / 443, 4000 1809 / 1683).
bool linear_wgrad_adam_pays(int64_t T, int64_t N, int64_t K, const float *dw) {
  if (K % 32 != 0 || (((uintptr_t)dw) & 127)) return false;
  if (T % 64 == 0) return true;
  GemmArgs g{N, K, T, nullptr, 1, N, nullptr, 1, K, nullptr, K, nullptr, nullptr, 3};
  return T >= 704 && fused_on_large_tiles(g);
}

static int pick_config(const GemmArgs &g) {
  const int f = forced_config();
  if (f >= 0) return f;
  const bool fused = g.c_mode == 3;
  if (fused && fused_on_large_tiles(g)) return kLdwLargeConfig;
  {
    std::lock_guard<std::mutex> lock(g_tuned_mutex);
    auto it = g_tuned.find(TuneKey(fused ? kFusedLayoutKey : layout_of(g), g.M, g.N, g.K));
    if (it != g_tuned.end()) return it->second;
  }
  return fused ? fused_config(g, nullptr) : heuristic_config(g);
}

static int launch_config(const GemmArgs &g, int config, hipStream_t s) {
  const bool akc = g.a_cs == 1, bkc = g.b_cs == 1;
  if (!g.c_mode && akc && bkc) return gemm_mfma_nt(g, config, s);
  if (!g.c_mode && akc && !bkc) return gemm_mfma_nn(g, config, s);
  if (g.c_mode && !akc && !bkc) return gemm_mfma_tn(g, config, s);
  return fail(TM_EINVAL, "gemm_mfma: operand layout not instantiated");
}

// ---- split reduction --------------------------------------------------------------------------------
// dx = dy W with a long reduction and few output tiles (the out-projection's input gradient: 2048 x 1536
// over 12288) fills a fraction of the chip.  With scratch from the caller the reduction is cut into parts
// whose 128x192 tiles make one pass of 512 blocks; the fp32 parts are added in part order and rounded once.
// The choice depends on the shape only, so results stay reproducible.
// With 256x192 tiles (the kernel with loader waves, one block per compute unit) when those make one pass of at least
// 192 blocks, else with 128x192 tiles, two blocks per unit.
static int splitk_parts(const GemmArgs &g, bool *large = nullptr) {
  if (large) *large = false;
  if (g.c_mode != 0 || g.bias || g.residual || !(g.a_cs == 1 && g.b_cs != 1)) return 1;
  const int64_t tiles = ceil_div(g.M, 128) * ceil_div(g.N, 192);
  if (tiles > 256 || g.K < 4096) return 1;
  const int64_t big = ceil_div(g.M, 256) * ceil_div(g.N, 192);
  int parts = (int)(256 / big);
  if (parts > 8) parts = 8;
  while (parts > 1 && g.K % (64 * parts) != 0) --parts;
  if (parts > 1 && big * parts >= 192) {
    if (large) *large = true;
    return parts;
  }
  parts = (int)(512 / tiles);
  if (parts > 8) parts = 8;
  while (parts > 1 && g.K % (64 * parts) != 0) --parts;
  return parts;
}

int64_t gemm_mfma_splitk_bytes(const GemmArgs &g) {
  const int parts = splitk_parts(g);
  return parts > 1 ? (int64_t)parts * g.M * g.N * 4 : 0;
}

// out[m, n] (bf16, row stride ldc) = sum over parts of part[p][m][n], eight columns per thread
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ part, int parts, int64_t M, int64_t N,
                                                            bf16 *__restrict__ out, int64_t ldc) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x, per_row = N / 8;
  if (idx >= M * per_row) return;
  const int64_t m = idx / per_row, n = (idx % per_row) * 8;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
  for (int q = 0; q < parts; ++q) {
    const float *src = part + ((int64_t)q * M + m) * N + n;
    const f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(src));
    const f32x4 b = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(src) + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) lo[e] += a[e], hi[e] += b[e];
  }
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (bf16)lo[e], o[4 + e] = (bf16)hi[e];
  *reinterpret_cast<bf16x8 *>(out + m * ldc + n) = o;
}

// Whether the split pays: its parts' product and the pass that adds them, against the unsplit product on the best tiles.
// The constants are fitted to 69 products of 1 to 4096 rows over 4096 to 20480: the choice is 1.2 % slower than the better of
// the two on them (geometric mean), where always splitting is 3 % slower and never splitting 14 %.  (2048 x 2048 over 4096: 58 us
// split, 30 unsplit on 128x128 tiles; 2048 x 512 over 4096: 29 against 17; 2048 x 1536 over 12288, the 175B shard's: 84 against 106;
// 3 x 64 over 8832: 24 against 27.)  The unsplit time is that of the tile configurations, also where the kernel for few tiles would
// have the product: that one, which the same call without scratch takes, is the faster of the two up to 256 rows (16 x 1024 over
// 8192 19.5 us, split 24.4; 64 x 1024 over 12288 28 and 32; 200 x 512 over 6144 13 and 21; 256 x 1024 over 8192 19 and 26).
static bool split_pays(const GemmArgs &g, int parts, bool large) {
  GemmArgs p = g;
  p.K = g.K / parts;
  const int c = large ? kLdwLargeConfig : 0;
  const int64_t nb = ceil_div(g.M, (int64_t)kConfigs[c].bm) * ceil_div(g.N, (int64_t)kConfigs[c].bn) * parts;
  const LayoutCost &k = kConfigs[c].cost[1];
  const double step_us = !large && nb > 256 ? k.pair : k.alone + k.fill * (nb < 256 ? (double)nb / 256.0 : 1.0);
  const double split_us = 1.25 * k.epi + (double)(p.K / 64) * step_us + 6.0 + (double)parts * g.M * g.N * 4 / 5e6;
  return 0.9 * split_us < config_us(g, heuristic_config(g), 1);
}

int gemm_mfma(const GemmArgs &g, hipStream_t s) {
  bool large = false;
  const int parts = splitk_parts(g, &large);
  if (parts > 1 && split_pays(g, parts, large) && g.splitk_scratch && g.splitk_bytes >= (int64_t)parts * g.M * g.N * 4 &&
      (((uintptr_t)g.splitk_scratch) & 15) == 0 && g.M * g.N * 4 < (1LL << 31) && forced_config() < 0) {
    GemmArgs p = g;
    p.C = g.splitk_scratch;
    p.ldc = g.N;
    p.c_mode = 2;
    p.k_splits = parts;
    if (int e = gemm_mfma_nn_partial(p, large, s)) return e;
    const int64_t groups = g.M * (g.N / 8);
    splitk_reduce_kernel<<<(unsigned)ceil_div(groups, (int64_t)256), 256, 0, s>>>((const float *)g.splitk_scratch, parts, g.M, g.N,
                                                                              (bf16 *)g.C, g.ldc);
    return check_launch("splitk_reduce");
  }
  if (forced_config() < 0 && gemm_mfma_small_pays(g)) return gemm_mfma_small(g, s);
  return launch_config(g, pick_config(g), s);
}

// Times every configuration and remembers the fastest for this layout and shape.  `variants` are n
// instances of the same product on different memory (say, the weights of different layers): the
// launches cycle through them, so that an operand that is cold in the real sequence is cold here too.
// The result buffers are overwritten several times; an accumulating product is timed in its
// overwriting form.  Synchronises the stream.
int gemm_mfma_tune(const GemmArgs *variants, int n, hipStream_t s) {
  if (n <= 0 || forced_config() >= 0) return TM_OK;
  std::vector<GemmArgs> v(variants, variants + n);
  for (GemmArgs &g : v) {
    if (!gemm_mfma_supported(g)) return TM_OK;
    if (g.M != v[0].M || g.N != v[0].N || g.K != v[0].K || layout_of(g) != layout_of(v[0]))
      return fail(TM_EINVAL, "gemm_mfma_tune: variants differ in shape or layout");
    g.bias = nullptr;
    g.residual = nullptr;
    if (g.c_mode == 1) g.c_mode = 2;
  }
  if (gemm_mfma_small_pays(v[0])) return TM_OK;  // takes none of the configurations
  const TuneKey key(layout_of(v[0]), v[0].M, v[0].N, v[0].K);
  {
    std::lock_guard<std::mutex> lock(g_tuned_mutex);
    if (g_tuned.count(key)) return TM_OK;
  }
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
    return fail(TM_ELAUNCH, "gemm_mfma_tune: cannot create events");
  float ms_of[kNumConfigs];
  int rc = TM_OK, turn = 0;
  for (int c = 0; c < kNumConfigs && rc == TM_OK; ++c) {
    ms_of[c] = 1e30f;
    rc = launch_config(v[turn++ % n], c, s);  // warm-up: code object load, clocks
    for (int r = 0; r < 3 && rc == TM_OK; ++r) {
      if (hipEventRecord(e0, s) != hipSuccess) rc = fail(TM_ELAUNCH, "gemm_mfma_tune: event record");
      if (rc == TM_OK) rc = launch_config(v[turn++ % n], c, s);
      if (rc == TM_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess))
        rc = fail(TM_ELAUNCH, "gemm_mfma_tune: event wait");
      float ms = 0.f;
      if (rc == TM_OK && hipEventElapsedTime(&ms, e0, e1) == hipSuccess && ms < ms_of[c]) ms_of[c] = ms;
    }
  }
  int best = 0;
  for (int c = 0; c < kNumConfigs; ++c)
    if (ms_of[c] < ms_of[best]) best = c;
  // the cost model's pick stays unless it loses by more than 1 %: keeps the choice stable against timer noise
  const int first = heuristic_config(v[0]);
  if (ms_of[first] <= 1.01f * ms_of[best]) best = first;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != TM_OK) return rc;
  if (getenv("TM_GEMM_TUNE_LOG")) {
    fprintf(stderr, "tune layout %d M=%lld N=%lld K=%lld:", layout_of(v[0]), (long long)v[0].M, (long long)v[0].N, (long long)v[0].K);
    for (int c = 0; c < kNumConfigs; ++c)
      fprintf(stderr, " %dx%dx%dx%d=%.4f%s", kConfigs[c].bm, kConfigs[c].bn, kConfigs[c].wgm, kConfigs[c].wgn, ms_of[c], c == best ? "*" : "");
    fprintf(stderr, "\n");
  }
  std::lock_guard<std::mutex> lock(g_tuned_mutex);
  g_tuned[key] = best;
  if (layout_of(v[0]) == 2) {
    float us[kNumConfigs];
    for (int c = 0; c < kNumConfigs; ++c) us[c] = ms_of[c] * 1e3f;
    g_tuned[TuneKey(kFusedLayoutKey, v[0].M, v[0].N, v[0].K)] = getenv("TM_GEMM_FUSED_ANY") ? best : fused_config(v[0], us);
  }
  return TM_OK;
}

}  // namespace tmk
