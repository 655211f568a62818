// LayerNorm / RMSNorm forward and backward, column reductions (bias and gain gradients).
// HBM-bound kernels: 16-byte accesses, fp32 arithmetic, wavefront shuffles for row sums.
#include <type_traits>

#include "columns.h"
#include "common.h"
#include "../../include/tm_ops.h"

namespace tmk {

constexpr int kNormThreads = 512;
constexpr int kNormMaxChunks = 4;  // 16-byte chunks per thread: hidden <= 512 * 4 * Vec::N

// Threads of a row.  TPR = 512: a block per row, for rows of more than 8 KB and for few rows.  Many shorter rows leave most
// of such a block idle and one small row in flight per block (4000 rows of 2 KB: 13.3 us forward, 21 backward; a wave per
// row: 6.4 and 11), so they take one wave (no barrier in the row sums), two or four, and a block holds 512 / TPR rows.  Where the
// line lies: norm_fwd_tpr, norm_bwd_tpr.
//
// Sum of two values over the TPR threads of this thread's row; red: 2 * 512 / 64 floats.
template <int TPR> __device__ __forceinline__ void row_sum2(float &a, float &b, float *red) {
  if constexpr (TPR == kNormThreads) {
    block_sum2<kNormThreads>(a, b, red);
  } else {
    a = wave_sum(a);
    b = wave_sum(b);
    if constexpr (TPR == 128) {
      constexpr int NW = kNormThreads / kWave;
      const int w = threadIdx.x / kWave;
      __syncthreads();  // protects `red` against the previous use
      if (threadIdx.x % kWave == 0) {
        red[w] = a;
        red[NW + w] = b;
      }
      __syncthreads();
      a = red[w & ~1] + red[w | 1];
      b = red[NW + (w & ~1)] + red[NW + (w | 1)];
    } else if constexpr (TPR == 256) {
      constexpr int NW = kNormThreads / kWave;
      const int w = threadIdx.x / kWave, w0 = w & ~3;
      __syncthreads();
      if (threadIdx.x % kWave == 0) {
        red[w] = a;
        red[NW + w] = b;
      }
      __syncthreads();
      a = (red[w0] + red[w0 + 1]) + (red[w0 + 2] + red[w0 + 3]);
      b = (red[NW + w0] + red[NW + w0 + 1]) + (red[NW + w0 + 2] + red[NW + w0 + 3]);
    }
  }
}

// ---------------------------------------------------------------------------------------
// forward: one block per token row; the row stays in registers between the passes.
// Every access goes through a per-row buffer descriptor (chunks past the row read as zero).
// COPY: x goes to `copy` as well, byte for byte (a form of its own: as a branch it cost the others up to 7 %).  A stage keeps
// its input so; a copy ahead of the norm was one more pass and launch (a step of the tiny preset 203.3 -> 200.5 us, the small
// bf16 layer's 0.8 % shorter).
// ---------------------------------------------------------------------------------------
template <typename T, int KIND, int NCH, bool COPY, int TPR = kNormThreads>
__global__ __launch_bounds__(kNormThreads) void norm_fwd_kernel(
    const T *__restrict__ x, const T *__restrict__ gain, const T *__restrict__ offset, T *__restrict__ out,
    float *__restrict__ mean_out, float *__restrict__ rstd_out, T *__restrict__ copy, int64_t rows, int h, float eps) {
  constexpr int VN = Vec<T>::N;
  __shared__ float red[2 * kNormThreads / kWave];
  const int tid = threadIdx.x % TPR;
  const int sub = TPR == kNormThreads ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / TPR);  // uniform over a wave
  const int64_t row = (int64_t)blockIdx.x * (kNormThreads / TPR) + sub;
  // a row past the end (several rows a block): reads as zero, nothing is written
  const bool in = TPR == kNormThreads || row < rows;
  const uint32_t row_bytes = in ? (uint32_t)h * sizeof(T) : 0u, width_bytes = (uint32_t)h * sizeof(T);
  const rsrc_t rx = make_rsrc(x + row * h, row_bytes), ro = make_rsrc(out + row * h, row_bytes);
  const rsrc_t rg = make_rsrc(gain, width_bytes), rf = make_rsrc(KIND == TM_NORM_LAYERNORM ? offset : gain, width_bytes);
  const int nchunk = h / VN;

  float vals[NCH][VN];
  float s1 = 0.f, s2 = 0.f;
  if constexpr (COPY) {
    typedef uint32_t raw4 __attribute__((ext_vector_type(4)));
    const rsrc_t rc = make_rsrc(copy + row * h, row_bytes);
    raw4 raw[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) raw[c] = __builtin_bit_cast(raw4, __builtin_amdgcn_raw_buffer_load_b128(rx, (tid + c * TPR) * 16u, 0, 0));
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      union { raw4 r; Vec<T> v; } u;
      u.r = raw[c];
      __builtin_amdgcn_raw_buffer_store_b128(raw[c], rc, (tid + c * TPR) * 16u, 0, 0);
#pragma unroll
      for (int i = 0; i < VN; ++i) vals[c][i] = to_f32(u.v.v[i]);
    }
  } else {
#pragma unroll
    for (int c = 0; c < NCH; ++c) buf_load_vec<T>(rx, (tid + c * TPR) * 16u, vals[c]);
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < VN; ++i) {
      s1 += vals[c][i];
      s2 += vals[c][i] * vals[c][i];
    }
  row_sum2<TPR>(s1, s2, red);
  float mu = 0.f, rstd;
  if (KIND == TM_NORM_LAYERNORM) {
    mu = s1 / h;
    float q = 0.f, dummy = 0.f;  // second pass over registers: sum of squared deviations
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const bool live = tid + c * TPR < nchunk;
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        const float dlt = vals[c][i] - mu;
        q += live ? dlt * dlt : 0.f;
      }
    }
    row_sum2<TPR>(q, dummy, red);
    rstd = 1.0f / sqrtf(q / h + eps);
  } else {
    rstd = 1.0f / sqrtf(s2 / h + eps);
  }
  if (tid == 0 && in) {
    if (mean_out) mean_out[row] = mu;
    rstd_out[row] = rstd;
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const uint32_t off = (tid + c * TPR) * 16u;
    float g[VN], o[VN], r[VN];
    buf_load_vec<T>(rg, off, g);
    if (KIND == TM_NORM_LAYERNORM) buf_load_vec<T>(rf, off, o);
#pragma unroll
    for (int i = 0; i < VN; ++i) {
      const float xh = (vals[c][i] - mu) * rstd;
      r[i] = (KIND == TM_NORM_LAYERNORM) ? xh * g[i] + o[i] : xh * g[i];
    }
    buf_store_vec<T>(ro, off, r);
  }
}

// ---------------------------------------------------------------------------------------
// backward: block b handles rows b, b+G, ...; each thread keeps the gain/offset gradient of
// its own columns in registers and writes one partial row per block at the end.
// partial layout: [G][3][h] fp32 (gain partials, offset partials, and with XSUM the column sums of the
// stored dx: the gradient of the bias of the linear map that produced x's residual input, which would
// otherwise cost one more pass over dx)
// ---------------------------------------------------------------------------------------
template <typename T, int KIND, int NCH, bool XSUM, int TPR = kNormThreads>
__global__ __launch_bounds__(kNormThreads) void norm_bwd_kernel(
    const T *__restrict__ dout, const T *__restrict__ x, const float *__restrict__ mean,
    const float *__restrict__ rstd, const T *__restrict__ gain, const T *dres, T *dx,
    float *__restrict__ partial, int64_t rows, int h) {
  constexpr int VN = Vec<T>::N;
  __shared__ float red[2 * kNormThreads / kWave];
  constexpr int RPB = kNormThreads / TPR;  // rows of a block at a time
  const int tid = threadIdx.x % TPR, sub = TPR == kNormThreads ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / TPR);
  const uint32_t row_bytes = (uint32_t)h * sizeof(T);
  const rsrc_t rg = make_rsrc(gain, row_bytes);
  float gacc[NCH][VN], oacc[NCH][VN], gn[NCH][VN], xacc[XSUM ? NCH : 1][VN];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    buf_load_vec<T>(rg, (tid + c * TPR) * 16u, gn[c]);
#pragma unroll
    for (int i = 0; i < VN; ++i) {
      gacc[c][i] = oacc[c][i] = 0.f;
      if (XSUM) xacc[c][i] = 0.f;
    }
  }
  // The loads of a block's NEXT row are in flight while it reduces and stores the current one (the raw 16-byte
  // chunks wait in registers): without that a block spends most of a row's time waiting for its three loads.
  typedef uint32_t raw4 __attribute__((ext_vector_type(4)));
  raw4 nw[NCH], nx[NCH], nr[NCH];
  auto fetch = [&](int64_t row) {
    const uint32_t bytes = TPR == kNormThreads || row < rows ? row_bytes : 0u;  // a row past the end reads as zeros
    const rsrc_t rd = make_rsrc(dout + row * h, bytes), rx = make_rsrc(x + row * h, bytes);
    const rsrc_t rr = make_rsrc(dres ? dres + row * h : dout, dres ? bytes : 0u);  // no residual: reads zeros
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const uint32_t off = (tid + c * TPR) * 16u;
      nw[c] = __builtin_bit_cast(raw4, __builtin_amdgcn_raw_buffer_load_b128(rd, off, 0, 0));
      nx[c] = __builtin_bit_cast(raw4, __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
      nr[c] = __builtin_bit_cast(raw4, __builtin_amdgcn_raw_buffer_load_b128(rr, off, 0, 0));
    }
  };
  auto unpack = [](raw4 raw, float (&out)[VN]) {
    union { raw4 r; Vec<T> v; } u;
    u.r = raw;
#pragma unroll
    for (int i = 0; i < VN; ++i) out[i] = to_f32(u.v.v[i]);
  };
  // all rows of a block advance together (barriers in the row sums): the loop runs on the block's first row
  const int64_t stride = (int64_t)gridDim.x * RPB;
  if ((int64_t)blockIdx.x * RPB < rows) fetch((int64_t)blockIdx.x * RPB + sub);
  for (int64_t row0 = (int64_t)blockIdx.x * RPB; row0 < rows; row0 += stride) {
    const int64_t row = row0 + sub;
    const bool in = TPR == kNormThreads || row < rows;
    const rsrc_t ro = make_rsrc(dx + row * h, in ? row_bytes : 0u);
    const float mu = KIND == TM_NORM_LAYERNORM && in ? mean[row] : 0.f;
    const float rs = in ? rstd[row] : 0.f;
    float w[NCH][VN], xh[NCH][VN], res[NCH][VN];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      unpack(nw[c], w[c]);
      unpack(nx[c], xh[c]);
      unpack(nr[c], res[c]);
    }
    if (row0 + stride < rows) fetch(row + stride);
    const int nchunk = h / VN;
    float sw = 0.f, swx = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const bool live = tid + c * TPR < nchunk;  // x reads as 0 past the row: xhat would be -mu*rs
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        const float d = w[c][i];
        const float xv = live ? (xh[c][i] - mu) * rs : 0.f;
        xh[c][i] = xv;
        w[c][i] = d * gn[c][i];
        gacc[c][i] += d * xv;
        oacc[c][i] += d;
        sw += w[c][i];
        swx += w[c][i] * xv;
      }
    }
    row_sum2<TPR>(sw, swx, red);
    const float mw = (KIND == TM_NORM_LAYERNORM) ? sw / h : 0.f;
    const float mwx = swx / h;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        res[c][i] += (w[c][i] - mw - xh[c][i] * mwx) * rs;
        if (XSUM) xacc[c][i] += to_f32(from_f32<T>(res[c][i]));  // the value as stored
      }
      buf_store_vec<T>(ro, (tid + c * TPR) * 16u, res[c]);
    }
  }
  if constexpr (RPB > 1) {  // the block's rows: their sums meet in LDS, added in row order, by the first TPR threads
    __shared__ float sums[kNormThreads * VN];
    auto join = [&](float (&v)[VN]) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < VN; ++i) sums[i * kNormThreads + threadIdx.x] = v[i];
      __syncthreads();
      if (sub == 0) {
#pragma unroll
        for (int i = 0; i < VN; ++i)
          for (int r = 1; r < RPB; ++r) v[i] += sums[i * kNormThreads + r * TPR + tid];
      }
    };
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      join(gacc[c]);
      join(oacc[c]);
      if constexpr (XSUM) join(xacc[c]);
    }
    if (sub != 0) return;
  }
  const rsrc_t rp = make_rsrc(partial + (int64_t)blockIdx.x * 3 * h, (uint32_t)h * 4u);
  const rsrc_t rq = make_rsrc(partial + (int64_t)blockIdx.x * 3 * h + h, (uint32_t)h * 4u);
  const rsrc_t rz = make_rsrc(partial + (int64_t)blockIdx.x * 3 * h + 2 * h, (uint32_t)h * 4u);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const uint32_t col = (tid + c * TPR) * VN;
#pragma unroll
    for (int v4 = 0; v4 < VN / 4; ++v4) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = gacc[c][v4 * 4 + i];
        b[i] = oacc[c][v4 * 4 + i];
      }
      buf_store_vec<float>(rp, (col + v4 * 4) * 4u, a);
      buf_store_vec<float>(rq, (col + v4 * 4) * 4u, b);
      if (XSUM) {
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = xacc[c][v4 * 4 + i];
        buf_store_vec<float>(rz, (col + v4 * 4) * 4u, z);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Column sums.  Up to nine of them share a launch: the partial rows of a layer's norms in the backward pass (gain, offset and dx
// sums of each), its bias gradients, or the second halves of these.  A launch of this kind takes 3 to 5 us whatever it adds up, and
// a layer with biases has seven or eight (together behind the last norm: 1.7 % of a step of the 6.7B shard, tiny preset 216 ->
// 203 us).
// ---------------------------------------------------------------------------------------
constexpr int kRowLanes = 16;  // row lanes of a block: 256 partial rows are four loads deep (four lanes: 7 us a launch, now 4.8)
constexpr int kMaxColumnTasks = 9;
struct ColumnTask {
  const void *src;  // [rows][ld], the first n columns of it
  float *out;
  int ld, rows, n, typed;  // typed: elements of the kernel's type, otherwise fp32
};
// MAX: tasks at most, 1, 3, 6 or 9 (looking one up is a chain of scalar loads and the table is a kernel argument: 0.8 of 11.5 us
// for one bias gradient of 12288 in a table of six)
template <int MAX> struct TaskTable {
  ColumnTask t[MAX];
  int first_block[MAX], count;
};
typedef TaskTable<kMaxColumnTasks> ColumnTasks;
template <int MAX> __device__ __forceinline__ int task_of_block(const TaskTable<MAX> &ts) {  // uniform over the block
  int i = 0;
#pragma unroll
  for (int k = 1; k < MAX; ++k)
    if (k < ts.count && (int)blockIdx.x >= ts.first_block[k]) i = k;
  return i;
}
template <int MAX> __device__ __forceinline__ int first_block_of(const TaskTable<MAX> &ts, int task) { return MAX == 1 ? 0 : ts.first_block[task]; }
template <typename E> __device__ __forceinline__ float column_rows(const E *src, int ld, int rows, int ry) {
  float s = 0.f;
  int r = ry;
  for (; r + 3 * kRowLanes < rows; r += 4 * kRowLanes) {  // four independent loads in flight per trip
    float a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = to_f32(src[(int64_t)(r + k * kRowLanes) * ld]);
#pragma unroll
    for (int k = 0; k < 4; ++k) s += a[k];
  }
  for (; r < rows; r += kRowLanes) s += to_f32(src[(int64_t)r * ld]);
  return s;
}
// out[c] (+)= sum_{r<rows} src[r*ld + c].  Block = 64 columns x 16 row lanes; lane y adds rows
// y, y+16, ... in ascending order, then the lane sums are added in lane order: a fixed order.
// BOTH: some tasks' rows are typed and some fp32; otherwise all are T (asking each costs a few percent of the short launches).
template <typename T, int MAX, bool BOTH>
__global__ __launch_bounds__(64 * kRowLanes) void column_sums_kernel(const TaskTable<MAX> ts, int accumulate) {
  __shared__ float sm[kRowLanes][64];
  const int task = task_of_block<MAX>(ts);
  const ColumnTask &t = ts.t[task];
  const int lane = threadIdx.x & 63, ry = threadIdx.x >> 6, c = ((int)blockIdx.x - first_block_of<MAX>(ts, task)) * 64 + lane;
  float s = 0.f;
  if (c < t.n) s = BOTH && !t.typed ? column_rows((const float *)t.src + c, t.ld, t.rows, ry) : column_rows((const T *)t.src + c, t.ld, t.rows, ry);
  sm[ry][lane] = s;
  __syncthreads();
  if (ry == 0 && c < t.n) {
    float sum = sm[0][lane];
#pragma unroll
    for (int k = 1; k < kRowLanes; ++k) sum += sm[k][lane];
    t.out[c] = accumulate ? t.out[c] + sum : sum;
  }
}

// First halves of column sums over many rows: block (column group, row group); task's out: partial [row groups][n]
constexpr int kColLanes = 64, kColRowsPerBlock = 4;
constexpr int kColsumDirectRows = 512;  // up to here in one launch, 32 rows a lane (256 rows of 256 to 1024: 3.5 us, two launches 5.0)

template <typename T, int MAX>
__global__ __launch_bounds__(kColLanes *kColRowsPerBlock) void colsum_partial_kernel(const TaskTable<MAX> ts, int rows_per_group) {
  constexpr int VN = Vec<T>::N;
  __shared__ float sm[kColRowsPerBlock][kColLanes * VN];
  const int task = task_of_block<MAX>(ts);
  const ColumnTask &t = ts.t[task];
  const T *dy = (const T *)t.src;
  const int lane = threadIdx.x % kColLanes, ry = threadIdx.x / kColLanes;
  const int col = (((int)blockIdx.x - first_block_of<MAX>(ts, task)) * kColLanes + lane) * VN;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_group;
  const int64_t r1 = (r0 + rows_per_group < t.rows) ? r0 + rows_per_group : t.rows;
  float acc[VN];
#pragma unroll
  for (int i = 0; i < VN; ++i) acc[i] = 0.f;
  if (col < t.n) {
    int64_t r = r0 + ry;
    for (; r + 3 * kColRowsPerBlock < r1; r += 4 * kColRowsPerBlock) {  // four rows in flight
      float v[4][VN];
#pragma unroll
      for (int k = 0; k < 4; ++k) load_vec<T>(dy + (r + k * kColRowsPerBlock) * t.ld + col, v[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < VN; ++i) acc[i] += v[k][i];
    }
    for (; r < r1; r += kColRowsPerBlock) {
      float v[VN];
      load_vec<T>(dy + r * t.ld + col, v);
#pragma unroll
      for (int i = 0; i < VN; ++i) acc[i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < VN; ++i) sm[ry][lane * VN + i] = acc[i];
  __syncthreads();
  if (ry == 0 && col < t.n) {
#pragma unroll
    for (int i = 0; i < VN; ++i) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < kColRowsPerBlock; ++k) s += sm[k][lane * VN + i];
      t.out[(int64_t)blockIdx.y * t.n + col + i] = s;
    }
  }
}

static int norm_bwd_blocks(int64_t T) { return (int)(T < 256 ? T : 256); }
// Threads of a row for width h (see the top of this file).  Few rows keep a block each, which leaves nothing to join: their
// time is one row's chain, and several rows a block add the join of their column sums to it.  Measured, a block a row
// against several rows a block, bf16, backward: 1024 wide, 64 rows 5.4 / 6.9 us, 192 rows 6.5 / 7.3, 256 rows 7.2 / 7.4 (with
// 300 rows some blocks get a second: 12 / 7.6); 512 wide (one chunk a lane, a shorter join) 32 rows 5.4 / 5.5, 96 rows 5.9 / 5.6.
// Forward (nothing to join): two waves a row 3.1 / 3.3 at up to 256 rows 2048 wide, one wave 3.0 / 2.8.
// Four waves a row (4 to 8 KB of it) have two chunks of a lane in flight instead of one, and two rows a block.  Forward, one
// row a block / two: 2048 rows of 4096 bf16 8.7 / 7.5 us, 8192 rows 25.4 / 21.8, 2048 of 1536 fp32 7.8 / 6.2.  Backward their
// join and registers cost, so only for rows of up to 5.5 KB, which leave more of a block idle, and from 1280 rows on, bf16
// 2304: 2391 of 1144 fp32 16.8 / 14.5, 7181 of 2480 bf16 44 / 39, but 1179 of 2176 12.8 / 13.7, 500 of 4096 11.8 / 13.1, 1641
// of 3968 17.3 / 17.8, 11941 of 3664 69.5 / 75.1 (1 to 10 % slower in most such sizes).
static int norm_fwd_tpr(int64_t T, int64_t h, int vn) {
  return h <= 2 * 64 * vn ? 64 : h <= 2 * 128 * vn && T > 256 ? 128 : h <= 2 * 256 * vn && T > 256 ? 256 : kNormThreads;
}
static int norm_bwd_tpr(int64_t T, int64_t h, int vn) {
  if (T <= (h <= 64 * vn ? 64 : 192)) return kNormThreads;
  return h <= 2 * 64 * vn ? 64 : h <= 2 * 128 * vn ? 128 : h <= 352 * vn && T > (vn == 8 ? 2304 : 1280) ? 256 : kNormThreads;
}
// blocks of the backward pass = partial rows: never more than norm_bwd_blocks, which sizes the scratch
static int norm_bwd_grid(int64_t T, int64_t h, int vn) {
  const int64_t groups = ceil_div(T, (int64_t)(kNormThreads / norm_bwd_tpr(T, h, vn)));
  return (int)(groups < 256 ? groups : 256);
}
// Row groups of a column sum, at most as many as a norm has partial rows (min(T, 256), which sizes the scratch): about 64
// rows each, and 32 groups where that would leave too few blocks.
static int colsum_groups(int64_t T) {
  if (T <= kColsumDirectRows) return 1;  // one launch, no partial rows
  return (int)(T <= 2048 ? 32 : T < 256 * 64 ? ceil_div(T, (int64_t)64) : 256);
}


// chunks per thread, rounded up to an instantiated count
static int pick_nch(int h, int vn) {
  const int need = (int)ceil_div(h / vn, kNormThreads);
  const int opts[] = {1, 2, 3, 4, 6, 8};
  for (int o : opts)
    if (need <= o) return o;
  return -1;
}
#define TM_NCH_SWITCH(nch, CALL)                    \
  switch (nch) {                                    \
    case 1: { constexpr int NCH = 1; CALL; } break; \
    case 2: { constexpr int NCH = 2; CALL; } break; \
    case 3: { constexpr int NCH = 3; CALL; } break; \
    case 4: { constexpr int NCH = 4; CALL; } break; \
    case 6: { constexpr int NCH = 6; CALL; } break; \
    default: { constexpr int NCH = 8; CALL; } break; \
  }

template <typename T, bool COPY>
static int norm_fwd_t(int kind, int64_t rows, int h, float eps, const void *x, const void *gain, const void *offset,
                      void *out, float *mean, float *rstd, void *copy, hipStream_t s) {
  const int nch = pick_nch(h, Vec<T>::N);
  g_last_kernel = "norm_fwd_kernel";
#define TM_NORM_FWD_NARROW(NCH, TPR)                                                                        \
  do {                                                                                                      \
    const unsigned grid = (unsigned)ceil_div(rows, (int64_t)(kNormThreads / TPR));                          \
    if (kind == TM_NORM_LAYERNORM)                                                                          \
      norm_fwd_kernel<T, TM_NORM_LAYERNORM, NCH, COPY, TPR><<<grid, kNormThreads, 0, s>>>(                  \
          (const T *)x, (const T *)gain, (const T *)offset, (T *)out, mean, rstd, (T *)copy, rows, h, eps); \
    else                                                                                                    \
      norm_fwd_kernel<T, TM_NORM_RMSNORM, NCH, COPY, TPR><<<grid, kNormThreads, 0, s>>>(                    \
          (const T *)x, (const T *)gain, nullptr, (T *)out, mean, rstd, (T *)copy, rows, h, eps);           \
    return check_launch("norm_fwd");                                                                        \
  } while (0)
  const int tpr = norm_fwd_tpr(rows, h, Vec<T>::N);
  if (tpr == 64 && h <= 64 * Vec<T>::N) TM_NORM_FWD_NARROW(1, 64);
  if (tpr == 64) TM_NORM_FWD_NARROW(2, 64);
  if (tpr == 128) TM_NORM_FWD_NARROW(2, 128);
  if (tpr == 256) TM_NORM_FWD_NARROW(2, 256);
#undef TM_NORM_FWD_NARROW
  if (kind == TM_NORM_LAYERNORM) {
    TM_NCH_SWITCH(nch, (norm_fwd_kernel<T, TM_NORM_LAYERNORM, NCH, COPY><<<dim3((unsigned)rows), kNormThreads, 0, s>>>(
                           (const T *)x, (const T *)gain, (const T *)offset, (T *)out, mean, rstd, (T *)copy, rows, h, eps)))
  } else {
    TM_NCH_SWITCH(nch, (norm_fwd_kernel<T, TM_NORM_RMSNORM, NCH, COPY><<<dim3((unsigned)rows), kNormThreads, 0, s>>>(
                           (const T *)x, (const T *)gain, nullptr, (T *)out, mean, rstd, (T *)copy, rows, h, eps)))
  }
  return check_launch("norm_fwd");
}

template <typename T, bool XSUM>
static int norm_bwd_t(int kind, int64_t rows, int h, const void *dout, const void *x, const float *mean,
                      const float *rstd, const void *gain, const void *dres, void *dx, float *partial, hipStream_t s) {
  const int G = norm_bwd_grid(rows, h, Vec<T>::N);
  const int nch = pick_nch(h, Vec<T>::N);
  g_last_kernel = "norm_bwd_kernel";
#define TM_NORM_BWD_NARROW(NCH, TPR)                                                                                   \
  do {                                                                                                                 \
    if (kind == TM_NORM_LAYERNORM)                                                                                     \
      norm_bwd_kernel<T, TM_NORM_LAYERNORM, NCH, XSUM, TPR><<<G, kNormThreads, 0, s>>>(                                \
          (const T *)dout, (const T *)x, mean, rstd, (const T *)gain, (const T *)dres, (T *)dx, partial, rows, h);     \
    else                                                                                                               \
      norm_bwd_kernel<T, TM_NORM_RMSNORM, NCH, XSUM, TPR><<<G, kNormThreads, 0, s>>>(                                  \
          (const T *)dout, (const T *)x, mean, rstd, (const T *)gain, (const T *)dres, (T *)dx, partial, rows, h);     \
    return check_launch("norm_bwd");                                                                                   \
  } while (0)
  const int tpr = norm_bwd_tpr(rows, h, Vec<T>::N);
  if (tpr == 64 && h <= 64 * Vec<T>::N) TM_NORM_BWD_NARROW(1, 64);
  if (tpr == 64) TM_NORM_BWD_NARROW(2, 64);
  if (tpr == 128) TM_NORM_BWD_NARROW(2, 128);
  if (tpr == 256) TM_NORM_BWD_NARROW(2, 256);
#undef TM_NORM_BWD_NARROW
  if (kind == TM_NORM_LAYERNORM) {
    TM_NCH_SWITCH(nch, (norm_bwd_kernel<T, TM_NORM_LAYERNORM, NCH, XSUM><<<G, kNormThreads, 0, s>>>(
                           (const T *)dout, (const T *)x, mean, rstd, (const T *)gain, (const T *)dres, (T *)dx,
                           partial, rows, h)))
  } else {
    TM_NCH_SWITCH(nch, (norm_bwd_kernel<T, TM_NORM_RMSNORM, NCH, XSUM><<<G, kNormThreads, 0, s>>>(
                           (const T *)dout, (const T *)x, mean, rstd, (const T *)gain, (const T *)dres, (T *)dx,
                           partial, rows, h)))
  }
  return check_launch("norm_bwd");
}

// appends a task of 64 (column_sums_kernel) or more columns a block; returns the blocks so far
static int add_task(ColumnTasks &ts, int blocks, int cols_per_block, const void *src, int64_t ld, int64_t rows, int64_t n, float *out, bool typed) {
  ts.first_block[ts.count] = blocks;
  ts.t[ts.count++] = ColumnTask{src, out, (int)ld, (int)rows, (int)n, typed};
  return blocks + (int)ceil_div(n, (int64_t)cols_per_block);
}
// go(table, MAX) on the smallest table that holds them
template <typename F> static void with_table(const ColumnTasks &ts, F &&go) {
  auto as = [&](auto max) {
    TaskTable<max()> t;
    for (int k = 0; k < max(); ++k) t.t[k] = ts.t[k], t.first_block[k] = ts.first_block[k];
    t.count = ts.count;
    go(t, max);
  };
  if (ts.count <= 1) as(std::integral_constant<int, 1>{});
  else if (ts.count <= 3) as(std::integral_constant<int, 3>{});
  else if (ts.count <= 6) as(std::integral_constant<int, 6>{});
  else as(std::integral_constant<int, kMaxColumnTasks>{});
}
static int launch_column_sums(int dtype, const ColumnTasks &ts, int blocks, int accumulate, hipStream_t s, const char *what) {
  bool typed = false, plain = false;  // (fp32: the same)
  for (int k = 0; k < ts.count; ++k) (ts.t[k].typed && dtype == TM_DTYPE_BF16 ? typed : plain) = true;
  auto go = [&](const auto &table, auto max) {
    if (typed && plain) column_sums_kernel<bf16, max(), true><<<(unsigned)blocks, 64 * kRowLanes, 0, s>>>(table, accumulate);
    else if (typed) column_sums_kernel<bf16, max(), false><<<(unsigned)blocks, 64 * kRowLanes, 0, s>>>(table, accumulate);
    else column_sums_kernel<float, max(), false><<<(unsigned)blocks, 64 * kRowLanes, 0, s>>>(table, accumulate);
  };
  with_table(ts, go);
  return check_launch(what);
}
// The sums over T rows of `count` matrices as tasks of the column_sums_kernel launch that follows: the matrices themselves
// where T is small, else their partial sums, which are enqueued here and go to `partial`.
static int add_column_sums(ColumnTasks &ts, int blocks, int dtype, int64_t T, const ColumnSum *sums, int count, float *partial, hipStream_t s) {
  if (T <= kColsumDirectRows) {
    for (int k = 0; k < count; ++k) blocks = add_task(ts, blocks, 64, sums[k].dy, sums[k].n, T, sums[k].n, sums[k].out, true);
    return blocks;
  }
  const int R = colsum_groups(T), vn = dtype == TM_DTYPE_BF16 ? 8 : 4;
  ColumnTasks first = {};
  int groups = 0;
  for (int k = 0; k < count; ++k) {
    groups = add_task(first, groups, kColLanes * vn, sums[k].dy, sums[k].n, T, sums[k].n, partial, true);
    blocks = add_task(ts, blocks, 64, partial, sums[k].n, R, sums[k].n, sums[k].out, false);
    partial += (int64_t)R * sums[k].n;
  }
  const dim3 grid((unsigned)groups, (unsigned)R);
  const int rows_per_group = (int)ceil_div(T, (int64_t)R);
  auto go = [&](const auto &table, auto max) {
    if (dtype == TM_DTYPE_BF16) colsum_partial_kernel<bf16, max()><<<grid, kColLanes * kColRowsPerBlock, 0, s>>>(table, rows_per_group);
    else colsum_partial_kernel<float, max()><<<grid, kColLanes * kColRowsPerBlock, 0, s>>>(table, rows_per_group);
  };
  with_table(first, go);
  return blocks;
}

}  // namespace tmk

using namespace tmk;

static int check_width(const char *what, int dtype, int64_t T, int64_t h) {
  if (dtype != TM_DTYPE_FP32 && dtype != TM_DTYPE_BF16) return fail(TM_EINVAL, "%s: unknown dtype %d", what, dtype);
  if (T <= 0 || h <= 0) return fail(TM_EINVAL, "%s: empty shape [%lld, %lld]", what, (long long)T, (long long)h);
  if (h % 8) return fail(TM_ESIZE, "%s: row width %lld is not a multiple of 8", what, (long long)h);
  if (T > 0x7fffffffLL / 8) return fail(TM_ESIZE, "%s: %lld rows exceed the supported range", what, (long long)T);
  return TM_OK;
}

extern "C" int64_t tm_op_reduce_scratch_bytes(int64_t T, int64_t width) {
  if (T <= 0 || width <= 0) return TM_EINVAL;
  const int64_t g1 = norm_bwd_blocks(T), g2 = colsum_groups(T);
  return (g1 > g2 ? g1 : g2) * width * (int64_t)sizeof(float);  // callers of the norm pass width = 3h
}

int tmk::norm_fwd_and_copy(int dtype, int kind, int64_t T, int64_t h, double eps, const void *x, const void *gain, const void *offset,
                           void *out, float *mean, float *rstd, void *copy, hipStream_t s) {
  if (int e = check_width("norm_fwd", dtype, T, h)) return e;
  if (kind != TM_NORM_LAYERNORM && kind != TM_NORM_RMSNORM) return fail(TM_EINVAL, "norm_fwd: unknown kind %d", kind);
  if (!x || !gain || !out || !rstd || (kind == TM_NORM_LAYERNORM && (!offset || !mean)))
    return fail(TM_EINVAL, "norm_fwd: NULL pointer");
  const int64_t hmax = (int64_t)kNormThreads * kNormMaxChunks * (dtype == TM_DTYPE_BF16 ? 8 : 4);
  if (h > hmax) return fail(TM_ESIZE, "norm_fwd: width %lld above the limit %lld", (long long)h, (long long)hmax);
  auto go = [&](auto copies) {
    constexpr bool COPY = copies();
    return dtype == TM_DTYPE_BF16 ? norm_fwd_t<bf16, COPY>(kind, T, (int)h, (float)eps, x, gain, offset, out, mean, rstd, copy, s)
                                  : norm_fwd_t<float, COPY>(kind, T, (int)h, (float)eps, x, gain, offset, out, mean, rstd, copy, s);
  };
  return copy ? go(std::true_type{}) : go(std::false_type{});
}

extern "C" int tm_op_norm_fwd(int dtype, int kind, int64_t T, int64_t h, double eps, const void *x, const void *gain,
                              const void *offset, void *out, float *mean, float *rstd, void *stream) {
  return norm_fwd_and_copy(dtype, kind, T, h, eps, x, gain, offset, out, mean, rstd, nullptr, (hipStream_t)stream);
}

static int norm_bwd_any(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean,
                        const float *rstd, const void *gain, const void *dres, void *dx, float *dgain, float *doffset,
                        float *dx_colsum, void *scratch, int accumulate, void *stream, const ColumnSum *sums = nullptr,
                        int count = 0, float *partial_sums = nullptr, const NormSums *earlier = nullptr, NormSums *later = nullptr) {
  if (int e = check_width("norm_bwd", dtype, T, h)) return e;
  if (kind != TM_NORM_LAYERNORM && kind != TM_NORM_RMSNORM) return fail(TM_EINVAL, "norm_bwd: unknown kind %d", kind);
  if (!dout || !x || !rstd || !gain || !dx || !dgain || !scratch || (kind == TM_NORM_LAYERNORM && (!mean || !doffset)))
    return fail(TM_EINVAL, "norm_bwd: NULL pointer");
  const int64_t hmax = (int64_t)kNormThreads * kNormMaxChunks * (dtype == TM_DTYPE_BF16 ? 8 : 4);
  if (h > hmax) return fail(TM_ESIZE, "norm_bwd: width %lld above the limit %lld", (long long)h, (long long)hmax);
  hipStream_t s = (hipStream_t)stream;
  float *partial = (float *)scratch;
  int e;
  if (dx_colsum)
    e = dtype == TM_DTYPE_BF16 ? norm_bwd_t<bf16, true>(kind, T, (int)h, dout, x, mean, rstd, gain, dres, dx, partial, s)
                               : norm_bwd_t<float, true>(kind, T, (int)h, dout, x, mean, rstd, gain, dres, dx, partial, s);
  else
    e = dtype == TM_DTYPE_BF16 ? norm_bwd_t<bf16, false>(kind, T, (int)h, dout, x, mean, rstd, gain, dres, dx, partial, s)
                               : norm_bwd_t<float, false>(kind, T, (int)h, dout, x, mean, rstd, gain, dres, dx, partial, s);
  if (e) return e;
  const int G = norm_bwd_grid(T, h, dtype == TM_DTYPE_BF16 ? Vec<bf16>::N : Vec<float>::N);
  const NormSums own{partial, G, h, {dgain, kind == TM_NORM_LAYERNORM ? doffset : nullptr, dx_colsum}};
  if (later) {
    *later = own;
    return TM_OK;
  }
  ColumnTasks ts = {};
  int blocks = 0;
  for (const NormSums *n : {&own, earlier})
    for (int k = 0; n && n->partial && k < 3; ++k)
      if (n->out[k]) blocks = add_task(ts, blocks, 64, n->partial + k * n->h, 3 * n->h, n->rows, n->h, n->out[k], false);
  if (count) blocks = add_column_sums(ts, blocks, dtype, T, sums, count, partial_sums, s);
  return launch_column_sums(dtype, ts, blocks, accumulate, s, "norm_bwd reduce");
}

int64_t tmk::column_sums_scratch_bytes(int64_t T, int64_t width) {
  return T <= kColsumDirectRows ? 0 : colsum_groups(T) * width * (int64_t)sizeof(float);
}

int tmk::norm_bwd_and_column_sums(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean,
                                  const float *rstd, const void *gain, const void *dres, void *dx, float *dgain, float *doffset,
                                  float *dx_colsum, void *scratch, const ColumnSum *sums, int count, void *partial_sums,
                                  const NormSums &earlier, int accumulate, hipStream_t s) {
  return norm_bwd_any(dtype, kind, T, h, dout, x, mean, rstd, gain, dres, dx, dgain, doffset, dx_colsum, scratch, accumulate, s, sums,
                      count, (float *)partial_sums, &earlier);
}

int64_t tmk::norm_bwd_partial_bytes(int dtype, int64_t T, int64_t h) {
  return (int64_t)norm_bwd_grid(T, h, dtype == TM_DTYPE_BF16 ? Vec<bf16>::N : Vec<float>::N) * 3 * h * (int64_t)sizeof(float);
}
int tmk::norm_bwd_rows(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x, const float *mean, const float *rstd,
                       const void *gain, const void *dres, void *dx, float *dgain, float *doffset, float *dx_colsum, void *scratch,
                       NormSums *later, hipStream_t s) {
  return norm_bwd_any(dtype, kind, T, h, dout, x, mean, rstd, gain, dres, dx, dgain, doffset, dx_colsum, scratch, 0, s, nullptr, 0, nullptr,
                      nullptr, later);
}

extern "C" int tm_op_norm_bwd(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x,
                              const float *mean, const float *rstd, const void *gain, const void *dres, void *dx,
                              float *dgain, float *doffset, void *scratch, int accumulate, void *stream) {
  return norm_bwd_any(dtype, kind, T, h, dout, x, mean, rstd, gain, dres, dx, dgain, doffset, nullptr, scratch, accumulate, stream);
}

extern "C" int tm_op_norm_bwd_colsum(int dtype, int kind, int64_t T, int64_t h, const void *dout, const void *x,
                                     const float *mean, const float *rstd, const void *gain, const void *dres, void *dx,
                                     float *dgain, float *doffset, float *dx_colsum, void *scratch, int accumulate,
                                     void *stream) {
  if (!dx_colsum) return fail(TM_EINVAL, "norm_bwd_colsum: NULL pointer");
  return norm_bwd_any(dtype, kind, T, h, dout, x, mean, rstd, gain, dres, dx, dgain, doffset, dx_colsum, scratch, accumulate, stream);
}

extern "C" int tm_op_bias_grad(int dtype, int64_t T, int64_t N, const void *dy, float *db, void *scratch,
                               int accumulate, void *stream) {
  if (int e = check_width("bias_grad", dtype, T, N)) return e;
  if (!dy || !db || !scratch) return fail(TM_EINVAL, "bias_grad: NULL pointer");
  hipStream_t s = (hipStream_t)stream;
  g_last_kernel = T <= kColsumDirectRows ? "column_sums_kernel" : "colsum_partial_kernel";
  const ColumnSum sum{dy, db, N};
  ColumnTasks ts = {};
  const int blocks = add_column_sums(ts, 0, dtype, T, &sum, 1, (float *)scratch, s);
  return launch_column_sums(dtype, ts, blocks, accumulate, s, "bias_grad");
}
