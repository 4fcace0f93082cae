// Row-wise (off-refresh) step of Periodic Row-wise Muon on gfx950.
//
// For every matrix: momentum update, RowNorm of the oriented momentum scaled
// by gamma, shape scale, decoupled weight decay and parameter write -- eq.
// (periodic-direction) with rho_t = 0, eq. (rownorm), Alg. 1 -- fused so that
// every element of G, M and W crosses HBM once (14 bytes per element for bf16
// W and G with fp32 M).
//
// Wide and square matrices (m <= n): an oriented row is a stored row.  One row
// is owned by TPR threads that keep its elements in registers across the
// sum-of-squares reduction (wave64 shuffles, then LDS across waves), so M is
// read once and written once.
//
// Tall matrices (m > n): an oriented row is a stored column, whose norm needs
// every stored row.  As in the sharded RowNorm of the paper's distributed
// execution (eq. sharded-tall-rownorm, App. "Correctness of sharded RowNorm"),
// row blocks play the role of the shards: pass 1 updates M and writes per-
// block column sums of squares, a finalize step reduces them in a fixed order
// and clamps after the square root, pass 2 writes W.
//
// All reductions have a fixed order, so results are bitwise reproducible.
#include <type_traits>

#include "prm_device.h"

namespace prm {

template <DType D> struct Store;
template <> struct Store<F32> { using T = float; };
template <> struct Store<BF16> { using T = uint16_t; };

// The element updates, with every rounding spelled out, so that a value does
// not depend on which kernel (aligned, ragged, small-set) it passes through in a
// later version.  Ragged rows (ALIGNED false) keep the forms their kernels have
// always had.
template <DType GD, bool ALIGNED>
__device__ __forceinline__ float new_momentum(float m, float g, const RwParams& p) {
  if constexpr (!ALIGNED && GD == F32) return fmaf(p.gcoef, g, p.beta * m);
  else return fmaf(p.beta, m, p.gcoef * g);
}
template <DType WD, bool ALIGNED>
__device__ __forceinline__ float new_weight(float w, float dv, const RwParams& p) {
  if constexpr (!ALIGNED && WD == BF16) return fmaf(-p.lr, dv, w * p.decay);
  else return fmaf(p.decay, w, -(p.lr * dv));
}

// Sum over the TPR threads that own one row.  All NT threads must call it.
template <int NT, int TPR>
__device__ __forceinline__ float row_sum(float v, float* red) {
  v = wave_sum(v);
  if constexpr (TPR == 64) {
    return v;
  } else {
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    constexpr int WPR = TPR / 64;
    const int first = (threadIdx.x / TPR) * WPR;
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < WPR; ++i) t += red[first + i];
    return t;
  }
}

// ---------------------------------------------------------------------------
// Wide rows in registers: NT threads per block, TPR threads per row, each
// thread owning NCH chunks of 8 consecutive elements.
// ---------------------------------------------------------------------------
template <int NT, int TPR, int NCH, DType WD, DType GD>
__device__ __forceinline__ void wide_row(const MatDesc& d, int64_t row, float* red, const RwParams& p) {
  using WT = typename Store<WD>::T;
  using GT = typename Store<GD>::T;
  const int64_t n = d.n;
  const int lt = threadIdx.x % TPR;
  const bool row_ok = row < d.m;

  const GT* G = reinterpret_cast<const GT*>(d.G) + row * n;
  float* M = d.M + row * n;
  WT* W = reinterpret_cast<WT*>(d.W) + row * n;

  float g[NCH][8], u[NCH][8], w[NCH][8];
  bool ok[NCH];
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    const int64_t e = (int64_t)(it * TPR + lt) * 8;
    ok[it] = row_ok && e < n;
    if (ok[it]) {
      VecNT<GT>::load8(G + e, g[it]);
      VecNT<float>::load8(M + e, u[it]);
      VecNT<WT>::load8(W + e, w[it]);
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    if (ok[it]) {
      const int64_t e = (int64_t)(it * TPR + lt) * 8;
#pragma unroll
      for (int k = 0; k < 8; ++k) u[it][k] = new_momentum<GD, true>(u[it][k], g[it][k], p);
      VecNT<float>::store8(M + e, u[it]);
      if (p.nesterov) {
#pragma unroll
        for (int k = 0; k < 8; ++k) u[it][k] = fmaf(p.beta, u[it][k], g[it][k]);
      }
      ss = it == 0 ? fmaf(u[it][0], u[it][0], u[it][1] * u[it][1])
                   : fmaf(u[it][1], u[it][1], fmaf(u[it][0], u[it][0], ss));
#pragma unroll
      for (int k = 2; k < 8; ++k) ss = fmaf(u[it][k], u[it][k], ss);
    }
  }
  ss = row_sum<NT, TPR>(ss, red);
  const float nu = fmaxf(sqrtf(ss), p.eps);
  const float kcoef = p.gamma * d.s * (1.0f / nu);
  float* const Dp = (p.write_d && d.D) ? d.D + row * n : nullptr;
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    if (ok[it]) {
      const int64_t e = (int64_t)(it * TPR + lt) * 8;
      float dv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        dv[k] = u[it][k] * kcoef;
        w[it][k] = new_weight<WD, true>(w[it][k], dv[k], p);
      }
      VecNT<WT>::store8(W + e, w[it]);
      if (Dp) VecNT<float>::store8(Dp + e, dv);
    }
  }
}

// Rows of any length and start, otherwise as above (TPR 64: a wave per row; 256:
// a block per row).  One pass with four elements an access instead of two sweeps of
// single elements; the last n % 8 elements are one each for the row's first
// threads.  The sum of squares is the one of the two-sweep kernel below, bit for
// bit: 256 partial sums over elements e, e + 256, ... (Kahan), for which the
// elements change hands through LDS (`x`: 8 TPR floats of the row).  HBM-bound; 60 M
// elements in rows of 3001, us in two sweeps / eight elements of a thread side by
// side, so that fp32 accesses left every other 16 bytes to the next one / now: 203 /
// 233 / 185 in fp32, 179 / 151 / 138 in bf16 (fp32 momentum).
template <int TPR, int NCH, DType WD, DType GD>
__device__ __forceinline__ void ragged_row(const MatDesc& d, int64_t row, float* x, float* red, const RwParams& p) {
  using WT = typename Store<WD>::T;
  using GT = typename Store<GD>::T;
  constexpr int SLOTS = 256 / TPR;  // partial sums per thread
  const int64_t n = d.n, n8 = n & ~(int64_t)7;
  const int lt = threadIdx.x % TPR;
  const bool row_ok = row < d.m;
  // a wave's LDS accesses run in order; rows of a block need its barrier
  auto exchange = [&]() __attribute__((always_inline)) {
    if constexpr (TPR == 64) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    else __syncthreads();
  };

  const GT* G = reinterpret_cast<const GT*>(d.G) + row * n;
  float* M = d.M + row * n;
  WT* W = reinterpret_cast<WT*>(d.W) + row * n;

  // Chunk `it` of the row is 8 TPR elements, two pieces of 4 to a thread (h), so that
  // every access is one span across the wave; gradients and weights stay as stored
  // until they are used (converted under the branch, each load would be waited for).
  typename RowIO<GT>::Raw g[NCH][2];
  typename RowIO<WT>::Raw w[NCH][2];
  float u[NCH][8];
  bool ok[NCH][2];
  auto at = [&](int it, int h) __attribute__((always_inline)) { return (int64_t)(2 * it + h) * (4 * TPR) + 4 * lt; };
#pragma unroll
  for (int it = 0; it < NCH; ++it)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t e = at(it, h);
      ok[it][h] = row_ok && e < n8;
      if (ok[it][h]) {
        g[it][h] = RowIO<GT>::load4(G + e);
        RowIO<float>::expand(RowIO<float>::load4(M + e), u[it] + 4 * h);
        w[it][h] = RowIO<WT>::load4(W + e);
      }
    }
  const int64_t et = n8 + lt;  // this thread's element of the row's ragged end
  const bool tail = row_ok && et < n;
  float gt = 0.f, ut = 0.f, wt = 0.f;
  if (tail) {
    gt = VecNT<GT>::load1(G + et);
    ut = VecNT<float>::load1(M + et);
    wt = VecNT<WT>::load1(W + et);
  }
  float ss[SLOTS], comp[SLOTS];
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) ss[j] = comp[j] = 0.f;
  auto add = [&](int j, float v) __attribute__((always_inline)) {
    const float y = fmaf(v, v, -comp[j]);
    const float t = ss[j] + y;
    comp[j] = (t - ss[j]) - y;
    ss[j] = t;
  };
#pragma unroll
  for (int it = 0; it < NCH; ++it) {
    if ((int64_t)it * TPR * 8 >= n8) break;  // the same for every thread of the row
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (ok[it][h]) {
        const int64_t e = at(it, h);
        float* const v = u[it] + 4 * h;
        float gv[4];
        RowIO<GT>::expand(g[it][h], gv);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = new_momentum<GD, false>(v[k], gv[k], p);
        RowIO<float>::store4(M + e, v);
        if (p.nesterov) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = fmaf(p.beta, v[k], gv[k]);
        }
        *reinterpret_cast<f32x4_t*>(x + h * 4 * TPR + 4 * lt) = f32x4_t{v[0], v[1], v[2], v[3]};
      }
    exchange();
    // elements it * 8 TPR + 256 k + (partial sum's number)
#pragma unroll
    for (int k = 0; k < 8 * TPR / 256; ++k)
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) {
        const int o = 256 * k + 64 * j + lt;
        if (row_ok && (int64_t)it * TPR * 8 + o < n8) add(j, x[o]);
      }
    exchange();
  }
  if (tail) {
    ut = new_momentum<GD, false>(ut, gt, p);
    VecNT<float>::store1(M + et, ut);
    if (p.nesterov) ut = fmaf(p.beta, ut, gt);
    x[lt] = ut;
  }
  exchange();
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) {
    const int o = (int)((64 * j + lt - n8) & 255);  // partial sum 64 j + lt takes element n8 + o
    if (row_ok && o < (int)(n - n8)) add(j, x[o]);
  }
  float sum;
  if constexpr (TPR == 64) {
    sum = 0.f;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) sum += wave_sum(ss[j]);
  } else {
    sum = block_sum<256>(ss[0], red);
  }
  const float nu = fmaxf(sqrtf(sum), p.eps);
  const float kcoef = p.gamma * d.s * (1.0f / nu);
  float* const Dp = (p.write_d && d.D) ? d.D + row * n : nullptr;
#pragma unroll
  for (int it = 0; it < NCH; ++it)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (ok[it][h]) {
        const int64_t e = at(it, h);
        float v[4], dv[4];
        RowIO<WT>::expand(w[it][h], v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          dv[k] = u[it][4 * h + k] * kcoef;
          v[k] = new_weight<WD, false>(v[k], dv[k], p);
        }
        RowIO<WT>::store4(W + e, v);
        if (Dp) RowIO<float>::store4(Dp + e, dv);
      }
  if (tail) {
    const float dv = ut * kcoef;
    VecNT<WT>::store1(W + et, new_weight<WD, false>(wt, dv, p));
    if (Dp) VecNT<float>::store1(Dp + et, dv);
  }
}

template <int NT, int TPR, int NCH, DType WD, DType GD, bool ALIGNED>
__global__ __launch_bounds__(NT) void rw_wide_kernel(const MatDesc* __restrict__ md,
                                                     const int32_t* __restrict__ seg_mat,
                                                     const int32_t* __restrict__ seg_start,
                                                     int32_t nseg, RwParams p) {
  constexpr int RPB = NT / TPR;
  __shared__ float red[NT / 64];
  __shared__ __attribute__((aligned(16))) float x[ALIGNED ? 4 : 8 * NT];
  const int seg = find_segment(seg_start, nseg, blockIdx.x);
  const int64_t row = (int64_t)((int)blockIdx.x - seg_start[seg]) * RPB + threadIdx.x / TPR;
  if constexpr (ALIGNED) wide_row<NT, TPR, NCH, WD, GD>(md[seg_mat[seg]], row, red, p);
  else ragged_row<TPR, NCH, WD, GD>(md[seg_mat[seg]], row, x + threadIdx.x / TPR * (8 * TPR), red, p);
}

// ---------------------------------------------------------------------------
// Wide rows too long for registers: one row per block, two sweeps; the second
// sweep re-reads the momentum this thread has just written.
// ---------------------------------------------------------------------------
template <DType WD, DType GD>
__global__ __launch_bounds__(256) void rw_generic_kernel(const MatDesc* __restrict__ md,
                                                         const int32_t* __restrict__ seg_mat,
                                                         const int32_t* __restrict__ seg_start,
                                                         int32_t nseg, RwParams p) {
  using WT = typename Store<WD>::T;
  using GT = typename Store<GD>::T;
  __shared__ float red[4];
  const int b = blockIdx.x;
  const int seg = find_segment(seg_start, nseg, b);
  const MatDesc& d = md[seg_mat[seg]];
  const int64_t n = d.n;
  const int64_t row = b - seg_start[seg];
  const GT* G = reinterpret_cast<const GT*>(d.G) + row * n;
  float* M = d.M + row * n;
  WT* W = reinterpret_cast<WT*>(d.W) + row * n;
  // a thread sums up to n / 256 squares (2^16 for the longest rows): with
  // compensation (Kahan) the sum stays within a few ulps
  float ss = 0.f, comp = 0.f;
  for (int64_t e = threadIdx.x; e < n; e += 256) {
    const float g = VecNT<GT>::load1(G + e);
    const float m = new_momentum<GD, false>(Vec<float>::load1(M + e), g, p);
    Vec<float>::store1(M + e, m);
    const float u = p.nesterov ? fmaf(p.beta, m, g) : m;
    const float y = fmaf(u, u, -comp);
    const float t = ss + y;
    comp = (t - ss) - y;
    ss = t;
  }
  ss = block_sum<256>(ss, red);
  const float nu = fmaxf(sqrtf(ss), p.eps);
  const float kcoef = p.gamma * d.s * (1.0f / nu);
  float* const Dp = (p.write_d && d.D) ? d.D + row * n : nullptr;
  for (int64_t e = threadIdx.x; e < n; e += 256) {
    const float m = Vec<float>::load1(M + e);
    const float u = p.nesterov ? fmaf(p.beta, m, VecNT<GT>::load1(G + e)) : m;
    const float dv = u * kcoef;
    VecNT<WT>::store1(W + e, new_weight<WD, false>(VecNT<WT>::load1(W + e), dv, p));
    if (Dp) Vec<float>::store1(Dp + e, dv);
  }
}

// ---------------------------------------------------------------------------
// Tall pass 1: momentum update and partial column sums of squares.
//
// n % 4 == 0: one block per tile of kTallRows (32) rows x 256 columns, and
// every thread loads its whole share once: wave w takes rows 8w .. 8w+7 of the
// tile, lane l the 4 columns 4l .. 4l+3, so each load or store instruction
// covers one contiguous 1 KB (fp32) or 512 B (bf16) span of a row.  Grids of
// such one-shot blocks stream HBM ~13% faster than blocks that loop over
// rows.  The four waves' column sums meet in LDS and wave 0 writes the
// tile's partial (fixed order).
// ---------------------------------------------------------------------------
constexpr int kTallRowsPerWave = kTallRows / 4;
static_assert(kTallRows % 4 == 0, "four waves share a tile's rows");

template <DType GD>
__device__ __forceinline__ void tall_stats(const MatDesc& d, const Item& it, float* red, const RwParams& p) {
  using GT = typename Store<GD>::T;
  constexpr int U = kTallRowsPerWave;
  const int64_t n = d.n;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t col = (int64_t)it.tn * 256 + 4 * lane;
  const int64_t r0 = (int64_t)it.tm * kTallRows + w * U;
  const bool ok = col < n;
  const GT* G = reinterpret_cast<const GT*>(d.G);
  float* M = d.M;
  float g[U][4], m[U][4];
#pragma unroll
  for (int q = 0; q < U; ++q) {
    if (ok && r0 + q < d.m) {
      const int64_t off = (r0 + q) * n + col;
      VecNT<GT>::load4(G + off, g[q]);
      VecNT<float>::load4(M + off, m[q]);
    }
  }
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < U; ++q) {
    if (ok && r0 + q < d.m) {
      const int64_t off = (r0 + q) * n + col;
#pragma unroll
      for (int k = 0; k < 4; ++k) m[q][k] = new_momentum<GD, true>(m[q][k], g[q][k], p);
      VecNT<float>::store4(M + off, m[q]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float u = p.nesterov ? fmaf(p.beta, m[q][k], g[q][k]) : m[q][k];
        acc[k] = fmaf(u, u, acc[k]);
      }
    }
  }
  *reinterpret_cast<f32x4_t*>(red + (w * 64 + lane) * 4) = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
  __syncthreads();
  if (w == 0 && ok) {
    float s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float* r = red + lane * 4 + k;
      s[k] = ((r[0] + r[256]) + r[512]) + r[768];
    }
    VecNT<float>::store4(d.colpart + (int64_t)it.tm * n + col, s);
  }
}

// n % 4 != 0: one column per thread, 256 columns and kTallRows rows per block,
// the loads of kBatch rows issued together: without a branch (rows past the last
// read the last again) and as stored (a 16-bit value converted under a branch is
// waited for there, row by row).  Whole step of bf16 weights and gradients, us, row by
// row / 8 / 16 rows: 4001 x 1003 42.6 / 25.1 / 22.2, 8001 x 3003 119 / 97 / 94.
// (16-byte accesses at any address, as the ragged rows use, ran at half the rate here:
// 8001 x 3003, 154 us against 64, where a wave's 1 KB span starts and ends inside a
// line at every row.)
constexpr int kBatch = 16;
static_assert(kTallRows % kBatch == 0, "whole batches");

template <DType GD>
__device__ __forceinline__ void tall_stats_scalar(const MatDesc& d, const Item& it, const RwParams& p) {
  using GT = typename Store<GD>::T;
  const int64_t n = d.n;
  const int64_t col = (int64_t)it.tn * 256 + threadIdx.x;
  if (col >= n) return;
  const int64_t r0 = (int64_t)it.tm * kTallRows;
  const int rows = (int)min((int64_t)kTallRows, d.m - r0);
  const GT* G = reinterpret_cast<const GT*>(d.G) + r0 * n + col;
  float* M = d.M + r0 * n + col;
  float acc = 0.f;
  for (int b = 0; b < rows; b += kBatch) {
    GT g[kBatch];
    float m[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      const uint32_t off = (uint32_t)min(b + q, rows - 1) * (uint32_t)n;  // < 32 * 2^24
      g[q] = VecNT<GT>::raw1(G + off);
      m[q] = Vec<float>::load1(M + off);
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q)
      if (b + q < rows) {
        const float gq = to_float(g[q]), v = new_momentum<GD, false>(m[q], gq, p);
        Vec<float>::store1(M + (uint32_t)(b + q) * (uint32_t)n, v);
        const float u = p.nesterov ? fmaf(p.beta, v, gq) : v;
        acc = fmaf(u, u, acc);
      }
  }
  Vec<float>::store1(d.colpart + (int64_t)it.tm * n + col, acc);
}

template <DType GD, bool ALIGNED>
__global__ __launch_bounds__(256) void rw_tall_stats_kernel(const MatDesc* __restrict__ md,
                                                            const Item* __restrict__ items,
                                                            RwParams p) {
  const Item it = items[blockIdx.x];
  if constexpr (ALIGNED) {
    __shared__ __attribute__((aligned(16))) float red[1024];
    tall_stats<GD>(md[it.mat], it, red, p);
  } else {
    tall_stats_scalar<GD>(md[it.mat], it, p);
  }
}

// Column norms of a tall matrix: fixed-order sum over row blocks, square root,
// then the clamp at eps (Alg. 2, row-wise branch: the clamp follows the square root).
__device__ __forceinline__ float col_inverse(const MatDesc& d, int64_t col, float eps) {
  // the loads of 16 row blocks are issued together and summed pairwise; the
  // group sums are accumulated with compensation (Kahan), so the error stays
  // at a few ulps however many row blocks a tall matrix has (fixed order)
  const float* cp = d.colpart + col;
  float s = 0.f, comp = 0.f;
  auto add = [&](float x) {
    const float y = x - comp;
    const float t = s + y;
    comp = (t - s) - y;
    s = t;
  };
  int rb = 0;
  for (; rb + 16 <= d.nrb; rb += 16) {
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = Vec<float>::load1(cp + (int64_t)(rb + k) * d.n);
#pragma unroll
    for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
      for (int k = 0; k < w; ++k) v[k] += v[k + w];
    add(v[0]);
  }
  for (; rb < d.nrb; ++rb) add(Vec<float>::load1(cp + (int64_t)rb * d.n));
  return 1.0f / fmaxf(sqrtf(s), eps);
}

// The same sums (bit for bit) with the loads of a column spread over eight
// threads: a block takes kFinCols columns, thread (g, c) sums the groups of 16
// row blocks g, g + 8, ... of column c, and the group sums are accumulated in
// order by one thread per column.  (One thread per column waited for its groups
// one after the other on a grid of n / 256 blocks.)
constexpr int kFinGroups = 64;  // group sums per round

__global__ __launch_bounds__(256) void rw_tall_finalize_kernel(const MatDesc* __restrict__ md,
                                                               const Item* __restrict__ items,
                                                               RwParams p) {
  __shared__ float part[kFinGroups][kFinCols];
  const Item it = items[blockIdx.x];
  const MatDesc& d = md[it.mat];
  const int c = threadIdx.x % kFinCols, lane = threadIdx.x / kFinCols;
  constexpr int LANES = 256 / kFinCols;
  const int64_t col = (int64_t)it.tn * kFinCols + c;
  const bool ok = col < d.n;
  const float* cp = d.colpart + col;
  const int groups = d.nrb / 16;
  float s = 0.f, comp = 0.f;
  auto add = [&](float x) {
    const float y = x - comp;
    const float t = s + y;
    comp = (t - s) - y;
    s = t;
  };
  for (int g0 = 0; g0 < groups; g0 += kFinGroups) {
    const int count = min(kFinGroups, groups - g0);
    if (ok)
      for (int g = lane; g < count; g += LANES) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = Vec<float>::load1(cp + (int64_t)((g0 + g) * 16 + k) * d.n);
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
          for (int k = 0; k < w; ++k) v[k] += v[k + w];
        part[g][c] = v[0];
      }
    __syncthreads();
    if (lane == 0)
      for (int g = 0; g < count; ++g) add(part[g][c]);
    __syncthreads();
  }
  if (lane == 0 && ok) {
    float v[16];
    const int rest = d.nrb - groups * 16;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < rest) v[k] = Vec<float>::load1(cp + (int64_t)(groups * 16 + k) * d.n);
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < rest) add(v[k]);
    Vec<float>::store1(d.colinv + col, 1.0f / fmaxf(sqrtf(s), p.eps));
  }
}

// Tall pass 2: D = gamma * s * U / nu_col and the parameter write, on the same
// one-shot tiles as pass 1 (ALIGNED: n % 4 == 0; otherwise one column per
// thread, the loads of BATCH rows issued together).  OWN_NORMS: the block sums its 256 columns' partials itself instead
// of reading what the finalize launch left (short matrices).
template <DType WD, DType GD, bool NEST, bool ALIGNED, bool OWN_NORMS, int BATCH>
__global__ __launch_bounds__(256) void rw_tall_apply_kernel(const MatDesc* __restrict__ md,
                                                            const Item* __restrict__ items,
                                                            RwParams p) {
  using WT = typename Store<WD>::T;
  using GT = typename Store<GD>::T;
  constexpr int U = kTallRowsPerWave;
  const Item it = items[blockIdx.x];
  const MatDesc& d = md[it.mat];
  const int64_t n = d.n;
  const float gs = p.gamma * d.s;
  const int64_t own = (int64_t)it.tn * 256 + threadIdx.x;  // this thread's column where it takes one
  if constexpr (ALIGNED) {
    __shared__ __attribute__((aligned(16))) float inv[OWN_NORMS ? 256 : 4];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t col = (int64_t)it.tn * 256 + 4 * lane;
    const bool ok = col < n;
    const int64_t r0 = (int64_t)it.tm * kTallRows + w * U;
    const GT* G = reinterpret_cast<const GT*>(d.G);
    const float* M = d.M;
    WT* W = reinterpret_cast<WT*>(d.W);
    float m[U][4], wv[U][4], g[NEST ? U : 1][4];
    auto load = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (r0 + q < d.m) {
          const int64_t off = (r0 + q) * n + col;
          VecNT<float>::load4(M + off, m[q]);
          VecNT<WT>::load4(W + off, wv[q]);
          if constexpr (NEST) VecNT<GT>::load4(G + off, g[q]);
        }
      }
      // keeps beta M + G behind the last load: under a row's branch it would wait
      // for that row (fp32, 16 of 2048 x 2040: 213 us against 200).  The small grids
      // that sum their own norms gain more from four blocks on a CU, which the
      // registers then do not allow.
      if constexpr (NEST && !OWN_NORMS) {
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
          for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(m[q][k]));
      }
    };
    float kc[4];
    if constexpr (OWN_NORMS) {
      if (ok) load();
      inv[threadIdx.x] = own < n ? col_inverse(d, own, p.eps) : 0.f;
      __syncthreads();
      if (!ok) return;
#pragma unroll
      for (int k = 0; k < 4; ++k) kc[k] = inv[4 * lane + k];
    } else {
      if (!ok) return;
      load();
      Vec<float>::load4(d.colinv + col, kc);  // shared by every tile of these columns: cached
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) kc[k] *= gs;
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (r0 + q < d.m) {
        const int64_t off = (r0 + q) * n + col;
        float dv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float u = m[q][k];
          if constexpr (NEST) u = fmaf(p.beta, m[q][k], g[q][k]);
          dv[k] = u * kc[k];
          wv[q][k] = new_weight<WD, true>(wv[q][k], dv[k], p);
        }
        VecNT<WT>::store4(W + off, wv[q]);
        if (p.write_d && d.D) VecNT<float>::store4(d.D + off, dv);
      }
    }
  } else {
    if (own >= n) return;
    const int64_t base = (int64_t)it.tm * kTallRows * n + own;
    const int rows = (int)min((int64_t)kTallRows, d.m - (int64_t)it.tm * kTallRows);
    const GT* G = reinterpret_cast<const GT*>(d.G) + base;
    const float* M = d.M + base;
    WT* W = reinterpret_cast<WT*>(d.W) + base;
    float* const D = (p.write_d && d.D) ? d.D + base : nullptr;
    float kc = 0.f;
    for (int b = 0; b < rows; b += BATCH) {
      float m[BATCH];
      WT wv[BATCH];
      GT g[NEST ? BATCH : 1];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) {
        const uint32_t off = (uint32_t)min(b + q, rows - 1) * (uint32_t)n;  // < 32 * 2^24
        m[q] = Vec<float>::load1(M + off);
        wv[q] = VecNT<WT>::raw1(W + off);
        if constexpr (NEST) g[q] = VecNT<GT>::raw1(G + off);
      }
      if (b == 0) kc = gs * (OWN_NORMS ? col_inverse(d, own, p.eps) : Vec<float>::load1(d.colinv + own));
#pragma unroll
      for (int q = 0; q < BATCH; ++q)
        if (b + q < rows) {
          float u = m[q];
          if constexpr (NEST) u = fmaf(p.beta, m[q], to_float(g[q]));
          const float dv = u * kc;
          const uint32_t off = (uint32_t)(b + q) * (uint32_t)n;
          VecNT<WT>::store1(W + off, new_weight<WD, false>(to_float(wv[q]), dv, p));
          if (D) Vec<float>::store1(D + off, dv);
        }
    }
  }
}

// ---------------------------------------------------------------------------
// The first pass of every matrix whose rows a block holds, in one launch (tall
// statistics first, then the wide rows): no launch has to drain before the next
// fills the chip.  The sums have the order of the separate kernels.
// ---------------------------------------------------------------------------
template <DType WD, DType GD>
__global__ __launch_bounds__(256) void rw_first_kernel(const MatDesc* __restrict__ md, const Item* __restrict__ items,
                                                       int32_t ntall, const int32_t* __restrict__ seg_mat,
                                                       const int32_t* __restrict__ seg_start, int32_t nseg,
                                                       RwParams p) {
  __shared__ __attribute__((aligned(16))) float lds[2048];
  __shared__ float red[4];
  if ((int)blockIdx.x < ntall) {
    const Item it = items[blockIdx.x];
    const MatDesc& d = md[it.mat];
    if (d.n % 4 == 0) tall_stats<GD>(d, it, lds, p);
    else tall_stats_scalar<GD>(d, it, p);
    return;
  }
  const int b = (int)blockIdx.x - ntall;
  const int seg = find_segment(seg_start, nseg, b);
  const MatDesc& d = md[seg_mat[seg]];
  const int64_t first = b - seg_start[seg], row = first * 4 + threadIdx.x / 64;
  if (d.n % 8 == 0) {
    if (d.n <= kWaveRow) wide_row<256, 64, 8, WD, GD>(d, row, red, p);
    else wide_row<256, 256, 8, WD, GD>(d, first, red, p);
  } else {
    if (d.n <= kRaggedWaveRow) ragged_row<64, 1, WD, GD>(d, row, lds + threadIdx.x / 64 * 512, red, p);
    else ragged_row<256, 8, WD, GD>(d, first, lds, red, p);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int NT, int TPR, DType WD, DType GD, bool AL>
static hipError_t wide_nch(int nch, const MatDesc* md, const int32_t* sm, const int32_t* ss,
                           int32_t nseg, int32_t nb, const RwParams& p, hipStream_t s) {
  dim3 g(nb), b(NT);
  switch (nch) {
    case 1: rw_wide_kernel<NT, TPR, 1, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 2: rw_wide_kernel<NT, TPR, 2, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 3: rw_wide_kernel<NT, TPR, 3, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 4: rw_wide_kernel<NT, TPR, 4, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 5: rw_wide_kernel<NT, TPR, 5, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 6: rw_wide_kernel<NT, TPR, 6, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 7: rw_wide_kernel<NT, TPR, 7, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    case 8: rw_wide_kernel<NT, TPR, 8, WD, GD, AL><<<g, b, 0, s>>>(md, sm, ss, nseg, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <DType WD, DType GD>
static hipError_t wide_tpr(int tpr, int nch, bool aligned, const MatDesc* md, const int32_t* sm,
                           const int32_t* ss, int32_t nseg, int32_t nb, const RwParams& p,
                           hipStream_t s) {
  switch (tpr) {
    case 64:
      if (aligned) return wide_nch<256, 64, WD, GD, true>(nch, md, sm, ss, nseg, nb, p, s);
      if (nch != 1) return hipErrorInvalidValue;
      rw_wide_kernel<256, 64, 1, WD, GD, false><<<dim3(nb), dim3(256), 0, s>>>(md, sm, ss, nseg, p);
      return hipGetLastError();
    case 256: return aligned ? wide_nch<256, 256, WD, GD, true>(nch, md, sm, ss, nseg, nb, p, s)
                             : wide_nch<256, 256, WD, GD, false>(nch, md, sm, ss, nseg, nb, p, s);
    case 512: return aligned ? wide_nch<512, 512, WD, GD, true>(nch, md, sm, ss, nseg, nb, p, s) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

// Calls f(weight type, gradient type) with the two as constants.
template <DType D> using DTypeC = std::integral_constant<DType, D>;
template <typename F>
static hipError_t by_types(DType wt, DType gt, F&& f) {
  if (wt == BF16 && gt == BF16) return f(DTypeC<BF16>{}, DTypeC<BF16>{});
  if (wt == BF16) return f(DTypeC<BF16>{}, DTypeC<F32>{});
  if (gt == BF16) return f(DTypeC<F32>{}, DTypeC<BF16>{});
  return f(DTypeC<F32>{}, DTypeC<F32>{});
}

hipError_t launch_rw_wide(int tpr, int nch, bool aligned, DType wt, DType gt, const MatDesc* md,
                          const int32_t* seg_mat, const int32_t* seg_start, int32_t nseg,
                          int32_t nblocks, const RwParams& p, hipStream_t s) {
  if (nblocks <= 0) return hipSuccess;
  return by_types(wt, gt, [&](auto w, auto g) {
    return wide_tpr<decltype(w)::value, decltype(g)::value>(tpr, nch, aligned, md, seg_mat, seg_start, nseg, nblocks, p, s);
  });
}

hipError_t launch_rw_first(DType wt, DType gt, const MatDesc* md, const Item* items, int32_t ntall,
                           const int32_t* seg_mat, const int32_t* seg_start, int32_t nseg, int32_t nblocks,
                           const RwParams& p, hipStream_t s) {
  if (ntall + nblocks <= 0) return hipSuccess;
  const dim3 grid(ntall + nblocks), b(256);
  return by_types(wt, gt, [&](auto w, auto g) {
    constexpr DType W = decltype(w)::value, G = decltype(g)::value;
    rw_first_kernel<W, G><<<grid, b, 0, s>>>(md, items, ntall, seg_mat, seg_start, nseg, p);
    return hipGetLastError();
  });
}

hipError_t launch_rw_generic(DType wt, DType gt, const MatDesc* md, const int32_t* rows_mat,
                             const int32_t* rows_start, int32_t nseg, int32_t nrows_total,
                             const RwParams& p, hipStream_t s) {
  if (nrows_total <= 0) return hipSuccess;
  dim3 g(nrows_total), b(256);
  if (wt == BF16 && gt == BF16) rw_generic_kernel<BF16, BF16><<<g, b, 0, s>>>(md, rows_mat, rows_start, nseg, p);
  else if (wt == BF16) rw_generic_kernel<BF16, F32><<<g, b, 0, s>>>(md, rows_mat, rows_start, nseg, p);
  else if (gt == BF16) rw_generic_kernel<F32, BF16><<<g, b, 0, s>>>(md, rows_mat, rows_start, nseg, p);
  else rw_generic_kernel<F32, F32><<<g, b, 0, s>>>(md, rows_mat, rows_start, nseg, p);
  return hipGetLastError();
}

hipError_t launch_rw_tall_stats(bool aligned, DType gt, const MatDesc* md, const Item* items,
                                int32_t nitems, const RwParams& p, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  dim3 g(nitems), b(256);
  if (aligned) {
    if (gt == BF16) rw_tall_stats_kernel<BF16, true><<<g, b, 0, s>>>(md, items, p);
    else rw_tall_stats_kernel<F32, true><<<g, b, 0, s>>>(md, items, p);
  } else {
    if (gt == BF16) rw_tall_stats_kernel<BF16, false><<<g, b, 0, s>>>(md, items, p);
    else rw_tall_stats_kernel<F32, false><<<g, b, 0, s>>>(md, items, p);
  }
  return hipGetLastError();
}

hipError_t launch_rw_tall_finalize(const MatDesc* md, const Item* items, int32_t nitems,
                                   const RwParams& p, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  rw_tall_finalize_kernel<<<dim3(nitems), dim3(256), 0, s>>>(md, items, p);
  return hipGetLastError();
}

hipError_t launch_rw_tall_apply(bool aligned, bool own_norms, bool one_row, DType wt, DType gt, const MatDesc* md,
                                const Item* items, int32_t nitems, const RwParams& p,
                                hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  return by_types(wt, gt, [&](auto w, auto g) {
    constexpr DType W = decltype(w)::value, G = decltype(g)::value;
    auto run = [&](auto nest, auto al, auto own, auto batch) {
      rw_tall_apply_kernel<W, G, decltype(nest)::value, decltype(al)::value, decltype(own)::value, decltype(batch)::value>
          <<<dim3(nitems), dim3(256), 0, s>>>(md, items, p);
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, kBatch> many{};
    auto own = [&](auto nest, auto al, auto batch) {
      own_norms ? run(nest, al, std::true_type{}, batch) : run(nest, al, std::false_type{}, batch);
    };
    auto al = [&](auto nest) {
      if (aligned) own(nest, std::true_type{}, many);
      else if (one_row) run(nest, std::false_type{}, std::false_type{}, one);
      else own(nest, std::false_type{}, many);
    };
    p.nesterov ? al(std::true_type{}) : al(std::false_type{});
    return hipGetLastError();
  });
}

}  // namespace prm
