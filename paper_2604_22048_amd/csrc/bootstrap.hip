// Multiplicative and additive shear bias by shape-noise cancellation with
// bootstrap errors (Section 3.5).  With the population parameters fixed the
// shear posterior of a galaxy resample that draws galaxy n c_n times is
//   ln P_b(g_p) = sum_n c_bn ell_n(g_p),
// so every resample of both datasets (+g and -g) is one dense product of the
// count matrix C [R x G] (row 0 all ones: every galaxy once; rows 1..B the
// resamples) with the per-galaxy log-marginal tables E+ and E- [P x G]:
//   Lp[r][p] = sum_n C[r][n] E[p][n],  p < 2P over [E+; E-].
// The product runs on the FP64 matrix cores (v_mfma_f64_16x16x4f64): a
// workgroup of 4 waves owns a 64 x 64 output tile (16 RT rows for few
// resamples) of one K split, its waves taking every fourth chunk of 8
// galaxies; the waves' sums are added through LDS and the partial tile is
// written; a second kernel adds the splits in order, forms each row's
// posterior mean of g on the grid, and m_r, c_r; a third takes the standard
// deviations over the resamples.  ell = -inf (a galaxy with no supported
// sample at that point) is carried as -1e300 so that a galaxy not drawn
// (c = 0) adds exactly 0.
#include <algorithm>

#include "bsi_kernels.h"

namespace bsi {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;     // output tile (rows r and columns p) per workgroup
constexpr int kKc = 8;        // galaxies per chunk: 2 per lane group, one MFMA step each
constexpr int kColTiles = kTile / 16;
constexpr double kNegBig = -1e300;
constexpr int kSplitTarget = 2304;   // workgroups of a product, about

// Vector loads from rows that are only element-aligned (odd G).
typedef int i32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 16-row tiles per workgroup tile for R rows: 4, or fewer where 4 would be padding.
inline int row_tiles(int R) { return R > 32 ? 4 : R > 16 ? 2 : 1; }

// One lane's operands of a chunk: 2 consecutive galaxies of each row and column.
template <int RT>
struct BiasChunk {
  i32x2u a[RT];
  f64x2u b[kColTiles];
};

// Partial products of one K split.  Grid: one workgroup per (output tile,
// split), the split fastest, so that with a multiple of 8 splits an XCD works
// on its own galaxies only; its workgroups go through them at about the same
// pace, row tiles of one column tile next to each other, so the XCD's L2 holds
// what they share.  out[z][r][p] for r < R, p < 2P.
//
// Bound by the FP64 matrix cores.  Lane (i, q) (i = lane % 16, q = lane / 16)
// holds galaxies 2 q and 2 q + 1 of row i and column i of a chunk, so the
// operands come from global memory as 8- and 16-byte loads without passing
// LDS, the next two chunks' in flight during this chunk's MFMAs (8 RT of 64
// cycles each), and no barrier stands between chunks.  501 x 2,178 x 10,000:
// 485 us, 45 TFLOP/s of the 62.7 that a large float64 product reaches on this
// card; staging 32 galaxies at a time through LDS between barriers took
// 1,359 us.
template <int RT>
__global__ void __launch_bounds__(256, 2)
    bias_gemm_kernel(const int32_t* __restrict__ counts, const double* __restrict__ ep,
                     const double* __restrict__ em, int G, int P, int R, int k_per_split, int n_split,
                     double* __restrict__ out) {
  __shared__ f64x4 xs[2][RT * kColTiles][kWave];   // two waves' accumulators on their way to the other two
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const int split = blockIdx.x % n_split, tile = blockIdx.x / n_split;
  const int n_rt = (R + 16 * RT - 1) / (16 * RT);
  const int r0 = (tile % n_rt) * 16 * RT, p0 = (tile / n_rt) * kTile;
  const int k_begin = split * k_per_split, k_end = min(G, k_begin + k_per_split);
  const int P2 = 2 * P;
  const int i = lane & 15, q = lane >> 4;
  // rows past R and columns past 2P read a valid one: their sums are not written
  const int32_t* arow[RT];
  const double* brow[kColTiles];
#pragma unroll
  for (int t = 0; t < RT; ++t) arow[t] = counts + (int64_t)max(min(r0 + 16 * t + i, R - 1) - 1, 0) * G;
#pragma unroll
  for (int t = 0; t < kColTiles; ++t) {
    const int p = min(p0 + 16 * t + i, P2 - 1);
    brow[t] = (p < P) ? ep + (int64_t)p * G : em + (int64_t)(p - P) * G;
  }
  const bool ones = r0 + i == 0;    // row 0 of the product: every galaxy once
  auto load = [&](int k) {
    BiasChunk<RT> c;
    const int n = k + 2 * q;
    if (k + kKc <= k_end) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
        c.a[t] = counts ? *reinterpret_cast<const i32x2u*>(arow[t] + n) : i32x2u{0, 0};
#pragma unroll
      for (int t = 0; t < kColTiles; ++t) c.b[t] = *reinterpret_cast<const f64x2u*>(brow[t] + n);
    } else {                          // the split's last galaxies: zeros past k_end
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bool in = n + j < k_end;
#pragma unroll
        for (int t = 0; t < RT; ++t) c.a[t][j] = in && counts ? arow[t][n + j] : 0;
#pragma unroll
        for (int t = 0; t < kColTiles; ++t) c.b[t][j] = in ? brow[t][n + j] : 0.0;
      }
    }
    return c;
  };
  f64x4 acc[RT][kColTiles];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < kColTiles; ++u) acc[t][u] = f64x4{0.0, 0.0, 0.0, 0.0};
  int k = k_begin + kKc * wave;
  BiasChunk<RT> c = load(k), c1 = load(k + 4 * kKc);
  for (; k < k_end; k += 4 * kKc) {
    const BiasChunk<RT> c2 = load(k + 8 * kKc);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      double a[RT], b[kColTiles];
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t] = (t == 0 && ones) ? 1.0 : (double)c.a[t][j];
      // -inf (and anything below) -> -1e300
#pragma unroll
      for (int u = 0; u < kColTiles; ++u) b[u] = (c.b[u][j] > kNegBig) ? c.b[u][j] : kNegBig;
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < kColTiles; ++u) acc[t][u] = mfma_f64(a[t], b[u], acc[t][u]);
    }
    c = c1;
    c1 = c2;
  }
  // waves 2, 3 -> 0, 1, then wave 1 -> 0
#pragma unroll
  for (int h = 2; h >= 1; h >>= 1) {
    __syncthreads();
    if (wave >= h && wave < 2 * h)
#pragma unroll
      for (int t = 0; t < RT * kColTiles; ++t) xs[wave - h][t][lane] = acc[t / kColTiles][t % kColTiles];
    __syncthreads();
    if (wave < h)
#pragma unroll
      for (int t = 0; t < RT * kColTiles; ++t) acc[t / kColTiles][t % kColTiles] += xs[wave][t][lane];
  }
  if (wave != 0) return;
  // D[i][j] of a 16 x 16 float64 tile sits in lane j + 16 (i % 4), element
  // i / 4 (rows interleaved across the lane groups, unlike the float32 form)
  double* o = out + (int64_t)split * R * P2;
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < kColTiles; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = r0 + 16 * t + q + 4 * e;
        const int p = p0 + 16 * u + i;
        if (r < R && p < P2) o[(int64_t)r * P2 + p] = acc[t][u][e];
      }
}

constexpr int kMeanThreads = 256;
constexpr int kAhead = 16;      // splits whose values are on their way together

// Fixed-order block sum of one value per thread (valid in thread 0).
__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = kMeanThreads / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double t = red[0];
  __syncthreads();
  return t;
}

__device__ __forceinline__ double block_max(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = kMeanThreads / 2; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  const double t = red[0];
  __syncthreads();
  return t;
}

// One workgroup per row r: the K splits added in order (read in batches: one
// after another they made a call of few resamples slower than a quarter of the
// splits did, 30,000 galaxies x 578 columns x 34 rows 264 us against 187, now
// 131), then for each of
// the two datasets the posterior mean of g on its grid (gpts, then gpts +
// 2 P; weights exp(ln P - max)),
// then m_r = (g+_1 - g-_1) / (2 |g|) - 1 and c_r = (g+_2 + g-_2) / 2.
__global__ void __launch_bounds__(kMeanThreads) bias_mean_kernel(const double* __restrict__ part,
                                                                 int n_split, int R, int P,
                                                                 const double* __restrict__ gpts,
                                                                 double g_abs, double* __restrict__ gmean,
                                                                 double* __restrict__ mc) {
  extern __shared__ double lp[];      // [2P]
  __shared__ double red[kMeanThreads];
  const int r = blockIdx.x, P2 = 2 * P;
  for (int p = threadIdx.x; p < P2; p += kMeanThreads) {
    double v = 0.0;
    const double* at = part + (int64_t)r * P2 + p;
    const int64_t step = (int64_t)R * P2;
    int s = 0;
    for (; s + kAhead <= n_split; s += kAhead, at += kAhead * step) {
      double t[kAhead];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) t[j] = at[j * step];
      __builtin_amdgcn_sched_barrier(0);     // the loads together, ahead of the adds
#pragma unroll
      for (int j = 0; j < kAhead; ++j) v += t[j];
    }
    for (; s < n_split; ++s, at += step) v += *at;
    lp[p] = v;
  }
  __syncthreads();
  double mean[2][2];
  for (int d = 0; d < 2; ++d) {
    const double* l = lp + d * P;
    const double* gd = gpts + 2 * (int64_t)d * P;
    double mx = -INFINITY;
    for (int p = threadIdx.x; p < P; p += kMeanThreads) mx = fmax(mx, l[p]);
    mx = block_max(mx, red);
    double w0 = 0.0, w1 = 0.0, w2 = 0.0;
    for (int p = threadIdx.x; p < P; p += kMeanThreads) {
      const double w = exp(l[p] - mx);
      w0 += w;
      w1 += w * gd[2 * p];
      w2 += w * gd[2 * p + 1];
    }
    w0 = block_sum(w0, red);
    w1 = block_sum(w1, red);
    w2 = block_sum(w2, red);
    mean[d][0] = w1 / w0;
    mean[d][1] = w2 / w0;
  }
  if (threadIdx.x == 0) {
    if (gmean) {
      gmean[2 * (int64_t)r] = mean[0][0];
      gmean[2 * (int64_t)r + 1] = mean[0][1];
      gmean[2 * ((int64_t)R + r)] = mean[1][0];
      gmean[2 * ((int64_t)R + r) + 1] = mean[1][1];
    }
    mc[2 * (int64_t)r] = (mean[0][0] - mean[1][0]) / (2.0 * g_abs) - 1.0;
    mc[2 * (int64_t)r + 1] = 0.5 * (mean[0][1] + mean[1][1]);
  }
}

// stats = {m_0, c_0, std(m_1..m_B), std(c_1..c_B)} (population standard
// deviations, two passes, fixed order); std 0 when B = 0.
__global__ void __launch_bounds__(kMeanThreads) bias_stats_kernel(const double* __restrict__ mc, int R,
                                                                  double* __restrict__ stats) {
  __shared__ double red[kMeanThreads];
  const int B = R - 1;
  double sd[2] = {0.0, 0.0};
  for (int q = 0; q < 2; ++q) {
    double s = 0.0;
    for (int b = 1 + threadIdx.x; b <= B; b += kMeanThreads) s += mc[2 * b + q];
    s = block_sum(s, red);
    const double mean = (B > 0) ? s / B : 0.0;
    double v = 0.0;
    for (int b = 1 + threadIdx.x; b <= B; b += kMeanThreads) {
      const double d = mc[2 * b + q] - mean;
      v += d * d;
    }
    v = block_sum(v, red);
    sd[q] = (B > 0) ? sqrt(v / B) : 0.0;
  }
  if (threadIdx.x == 0) {
    stats[0] = mc[0];
    stats[1] = mc[1];
    stats[2] = sd[0];
    stats[3] = sd[1];
  }
}

}  // namespace

BiasPlan bias_plan(int G, int P, int n_boot) {
  BiasPlan b;
  b.R = n_boot + 1;
  const int tiles = ((2 * P + kTile - 1) / kTile) * ((b.R + 16 * row_tiles(b.R) - 1) / (16 * row_tiles(b.R)));
  // about kSplitTarget workgroups (4.5 rounds of two per compute unit, so that
  // the last round is a small share), each with at least four chunks per wave;
  // from 8 splits on a multiple of 8, one XCD's galaxies each
  int splits = std::max(1, std::min((kSplitTarget + tiles / 2) / tiles, G / (16 * kKc)));
  if (splits >= 8) splits = splits / 8 * 8;
  b.k_per_split = ((G + splits - 1) / splits + kKc - 1) / kKc * kKc;
  b.n_split = std::max(1, (G + b.k_per_split - 1) / b.k_per_split);
  b.partial_doubles = (size_t)b.n_split * b.R * 2 * P;
  return b;
}

size_t bias_partial_bound(int P, int n_boot) {
  // n_split tiles <= kSplitTarget + tiles, a tile at most 64 x 64 values
  const size_t rows = (size_t)(n_boot + kTile) / kTile * kTile, cols = (size_t)(2 * P + kTile - 1) / kTile * kTile;
  return (size_t)kSplitTarget * kTile * kTile + rows * cols;
}

size_t bias_mean_lds_bytes(int P) { return sizeof(double) * 2 * (size_t)P; }

hipError_t launch_bias(const BiasPlan& b, const int32_t* counts, const double* ep, const double* em,
                       int G, int P, const double* gpts, double g_abs, double* partial, double* gmean,
                       double* mc, double* stats, hipStream_t s) {
  const int rt = row_tiles(b.R);
  const int tiles = ((2 * P + kTile - 1) / kTile) * ((b.R + 16 * rt - 1) / (16 * rt));
  auto gemm = rt == 4 ? bias_gemm_kernel<4> : rt == 2 ? bias_gemm_kernel<2> : bias_gemm_kernel<1>;
  hipLaunchKernelGGL(gemm, dim3(tiles * b.n_split), dim3(256), 0, s, counts, ep, em, G, P, b.R,
                     b.k_per_split, b.n_split, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = bias_mean_lds_bytes(P);
  (void)hipFuncSetAttribute((const void*)bias_mean_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
  hipLaunchKernelGGL(bias_mean_kernel, dim3(b.R), dim3(kMeanThreads), lds, s, partial, b.n_split, b.R,
                     P, gpts, g_abs, gmean, mc);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bias_stats_kernel, dim3(1), dim3(kMeanThreads), 0, s, mc, b.R, stats);
  return hipGetLastError();
}

}  // namespace bsi
