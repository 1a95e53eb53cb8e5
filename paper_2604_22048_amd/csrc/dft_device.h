// Forward DFT of a stamp in LDS at the half-plane bins of the k-space
// likelihood, as two dense products on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32), result in slot order in LDS:
//   pass A  Q[v][x] = sum_y d[y][x] e^{-i k_v y'}      (rows v = 0..h; -h for
//                                                       the last row of even N)
//   pass B  D[v][u] = sum_x Q[v][x] e^{-i k_u x'}      (the N DFT columns u)
// with pixel centres at x' = x - (N-1)/2.  Both passes read one table of DFT
// factors e^{-i k_f p'}, f = 0..h, laid out as the MFMA operands are held
// (blocks of 16 frequencies, per K step one 8-byte LDS read per lane, the lanes
// consecutive); pass B takes the columns +u and -u together, the factors of
// one being the conjugates of the other's.  The tables are filled once per
// device and copied into LDS with the stamp.  (Looked up from a 2N-entry
// twiddle table instead, the factors' random LDS reads and index arithmetic
// took longer than the products; read from L2, their latency did.)
#pragma once

#include <algorithm>

#include "bsi_kernels.h"
#include "kspace.h"

namespace bsi {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct DftDims {
  int h, nrow;         // frequencies 0..h (rows of Q and D)
  int nrb, ncb;        // 16-row blocks of frequencies, 16-column blocks of pixels
  int steps;           // K steps of 4 pixels
  int ldQ;             // row stride of Q: 4 mod 8 float2, so that 16 rows' reads fall on all banks
  int last;            // frequencies of the last block
  int nblk;            // table blocks: nrb, and where last <= 8 one of last's +f (lanes 0..7) and -f (8..15)
};

__host__ __device__ constexpr DftDims dft_dims(int N) {
  DftDims d{};
  d.h = N / 2;
  d.nrow = d.h + 1;
  d.nrb = (d.nrow + 15) / 16;
  d.ncb = (N + 15) / 16;
  d.steps = (N + 3) / 4;
  d.ldQ = 4 * d.steps + (d.steps % 2 ? 0 : 4);
  d.last = d.nrow - 16 * (d.nrb - 1);
  d.nblk = d.nrb + (d.last <= 8 ? 1 : 0);
  return d;
}

// Table entries of one stamp side: [nblk][steps][64].
__host__ __device__ constexpr int dft_tab_len(int N) {
  const DftDims d = dft_dims(N);
  return d.nblk * d.steps * 64;
}

// Offset of side N's entries among those of sides 8..128 (N = 129: the total).
__host__ __device__ constexpr int dft_tab_off(int N) {
  int o = 0;
  for (int n = 8; n < N; ++n) o += dft_tab_len(n);
  return o;
}

// {k_u, sinc(u / N)} pairs, u = 0..h, of one side.
constexpr int kSincLen = 65;

// Units of work of the passes: pairs of row blocks by column blocks (A), row
// blocks by table blocks (B).  A wave holds up to U of either in registers.
__host__ __device__ constexpr int dft_units(int N) {
  const DftDims d = dft_dims(N);
  const int a = (d.nrb + 1) / 2 * d.ncb, b = d.nrb * d.nblk - (d.nblk > d.nrb ? d.nrb : 0);
  return a > b ? a : b;
}

// Units a wave of at most 8 holds: one, two, or four (128 px).
__host__ __device__ constexpr int dft_per_wave(int N) { return dft_units(N) <= 8 ? 1 : dft_units(N) <= 16 ? 2 : 4; }

// Stamps whose table exceeds the LDS beside the rest: it is read from memory.
__host__ __device__ constexpr bool dft_big(int N) { return dft_per_wave(N) > 2; }

// K steps whose operands are on their way while others are multiplied (a step's
// MFMAs take 64 to 256 cycles, LDS reads about 100, the tables from L2, for
// stamps whose tables exceed LDS, several hundred).  The last ones read up to
// kAhead steps past the operands' end, within the workgroup's LDS and the
// tables' padding, and are not used.
constexpr int kAhead = 4;

// LDS of stamp_dft: one region that holds the stamp (float, zero rows up to a
// whole K step), then Q, then D (float2, slot order), each pass keeping its
// results in registers until every wave has read its operands; the table
// (whole, padded); the rows' slot bases.
struct DftLds {
  size_t r, tab, rows;     // bytes of each
};

__host__ __device__ inline DftLds dft_lds(int N, const SlotPlan& sp) {
  const DftDims d = dft_dims(N);
  // steps read ahead past the stamp fall into what follows it, the table above
  // all, or without one (dft_big) into the region itself
  const size_t a = sizeof(float) * ((size_t)4 * (d.steps + (dft_big(N) ? kAhead : 0)) * N + 64);
  const size_t q = sizeof(float2) * ((size_t)d.nrow * d.ldQ + 4 * kAhead), b = sizeof(float2) * (size_t)sp.nbins;
  const size_t m = a > q ? a : q;
  return {((m > b ? m : b) + 15) & ~(size_t)15, sizeof(float2) * ((size_t)d.nblk * d.steps + kAhead) * 64,
          sizeof(int) * (size_t)d.nrb * 16};
}

// Pair-slot of (0, v) for every row v (16 entries per row block).
__device__ __forceinline__ void dft_row_bases(int N, const SlotPlan& sp, int* rows) {
  const int npc = pair_cols(N);
  for (int v = threadIdx.x; v < 16 * dft_dims(N).nrb; v += blockDim.x) rows[v] = v / sp.R * sp.P * 64 + v % sp.R * npc;
}

__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(kWaitVmcnt0); }

// Load stamp `data` (minus `model`, both at the stamp's first pixel) into d and
// zero its rows up to a whole K step; the caller synchronises.  Returns this
// thread's part of sum (data - model)^2.  Without a model the pixels (and
// whatever else the wave has under way) go straight into LDS.
__device__ __forceinline__ double load_stamp(int N, const float* __restrict__ data,
                                             const double* __restrict__ model, float* d) {
  const int n = N * N, full = 4 * ((N + 3) / 4) * N;
  const int lane = lane_id(), w0 = __builtin_amdgcn_readfirstlane(threadIdx.x - lane);
  double sq = 0.0;
  if (model) {
#pragma unroll 4
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
      const double x = (double)data[t] - model[t];
      d[t] = (float)x;
      sq = fma(x, x, sq);
    }
    for (int t = n + threadIdx.x; t < full; t += blockDim.x) d[t] = 0.f;
    wait_loads();
    return sq;
  }
  // the last transfer is ragged: its idle lanes repeat the last pixel past the
  // stamp's end, where the same wave then writes the zeros
  int t = w0;
  for (; t < n; t += blockDim.x)
    __builtin_amdgcn_global_load_lds(data + min(t + lane, n - 1), d + t, 4, 0, 0);
  wait_loads();
  if (t - (int)blockDim.x <= n - 1 && t - (int)blockDim.x + kWave >= n && w0 < n)
    for (int z = n + lane; z < full; z += kWave) d[z] = 0.f;
  return sq;
}

// Touch a stamp's memory (one load per 128-byte line of its own range) so that it
// is in L2 when load_stamp comes for it; consumed by touch_done.
__device__ __forceinline__ float touch_stamp(int N, const float* __restrict__ data) {
  const int t = 32 * threadIdx.x;
  return t < N * N ? data[t] : 0.f;
}

__device__ __forceinline__ void touch_done(float x) { asm volatile("" ::"v"(x)); }

// Copy a table of `entries` (a multiple of 64) into LDS, 16 bytes per lane (with
// the stamp's wait).
__device__ __forceinline__ void load_table(const float2* __restrict__ tab, float2* t, int entries) {
  const int lane = lane_id(), w0 = __builtin_amdgcn_readfirstlane(threadIdx.x - lane);
  // 64 entries are half a wave's transfer; an odd count ends in the padding
  for (int i = 2 * w0; i < entries; i += 2 * blockDim.x)
    __builtin_amdgcn_global_load_lds(tab + i + 2 * lane, t + i, 16, 0, 0);
}

// Pass A for RB row blocks from rb0 and column block cb: one stamp operand per
// step for 2 RB MFMAs.
template <int RB>
__device__ __forceinline__ void dft_pass_a(int N, const DftDims& g, const float* d, const float2* tab, int rb0, int cb,
                                           f32x4* qr, f32x4* qi) {
  const int lane = lane_id(), li = lane & 15, lk = lane >> 4;
  const float* dp = d + lk * N + cb * 16 + li;
  const float2* ta[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    ta[r] = tab + (rb0 + r) * g.steps * 64 + lane;
    qr[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    qi[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float2 w[kAhead][RB];
  float b[kAhead];
  auto load = [&](int i) {
#pragma unroll
    for (int r = 0; r < RB; ++r) w[i][r] = ta[r][i * 64];
    b[i] = dp[i * 4 * N];
  };
  auto mul = [&](int i) {
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      qr[r] = mfma16x16x4(w[i][r].x, b[i], qr[r]);
      qi[r] = mfma16x16x4(w[i][r].y, b[i], qi[r]);
    }
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i) load(i);
  int s = 0;
  for (; s + kAhead <= g.steps; s += kAhead) {
#pragma unroll
    for (int r = 0; r < RB; ++r) ta[r] += kAhead * 64;
    dp += kAhead * 4 * N;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      mul(i);
      load(i);
    }
  }
#pragma unroll
  for (int i = 0; i < kAhead - 1; ++i)
    if (s + i < g.steps) mul(i);
}

// Pass A's results to their places in Q.
__device__ __forceinline__ void dft_store_q(int N, const DftDims& g, float2* Q, int rb, int cb, f32x4 qr, f32x4 qi) {
  const int lane = lane_id(), x = cb * 16 + (lane & 15);
  if (x >= 4 * g.steps) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = rb * 16 + 4 * (lane >> 4) + j;
    if (row < g.nrow) Q[row * g.ldQ + x] = x < N ? make_float2(qr[j], qi[j]) : make_float2(0.f, 0.f);
  }
}

// Pass B for row block rb and the DFT columns of table block cb: +u and -u of
// its 16 frequencies (PAIR), or the merged block's own columns; one Q operand
// and one factor per step for 8 or 4 MFMAs.
template <bool PAIR>
__device__ __forceinline__ void dft_pass_b(const DftDims& g, const float2* Q, const float2* tab, int rb, int cb,
                                           f32x4* dr, f32x4* di) {
  constexpr int CB = PAIR ? 2 : 1;
  const int lane = lane_id(), li = lane & 15, lk = lane >> 4;
  // rows past the last read it again: their sums are not kept
  const float2* qp = Q + min(rb * 16 + li, g.nrow - 1) * g.ldQ + lk;
  const float2* tb = tab + cb * g.steps * 64 + lane;
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    dr[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    di[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float2 w[kAhead], q[kAhead];
  auto load = [&](int i) {
    w[i] = tb[i * 64];
    q[i] = qp[i * 4];
  };
  auto mul = [&](int i) {
    dr[0] = mfma16x16x4(q[i].x, w[i].x, dr[0]);
    di[0] = mfma16x16x4(q[i].x, w[i].y, di[0]);
    if (PAIR) {
      dr[CB - 1] = mfma16x16x4(q[i].x, w[i].x, dr[CB - 1]);
      di[CB - 1] = mfma16x16x4(-q[i].x, w[i].y, di[CB - 1]);
    }
    dr[0] = mfma16x16x4(-q[i].y, w[i].y, dr[0]);
    di[0] = mfma16x16x4(q[i].y, w[i].x, di[0]);
    if (PAIR) {
      dr[CB - 1] = mfma16x16x4(q[i].y, w[i].y, dr[CB - 1]);
      di[CB - 1] = mfma16x16x4(q[i].y, w[i].x, di[CB - 1]);
    }
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i) load(i);
  int s = 0;
  for (; s + kAhead <= g.steps; s += kAhead) {
    tb += kAhead * 64;
    qp += kAhead * 4;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      mul(i);
      load(i);
    }
  }
#pragma unroll
  for (int i = 0; i < kAhead - 1; ++i)
    if (s + i < g.steps) mul(i);
}

// sqrt w = lambda^-1/2 of DFT mode (u, v >= 0 or -h), ps in FFT order (NULL: white).
__device__ __forceinline__ float sqrt_weight(const float* __restrict__ ps, int N, int u, int v) {
  return ps ? (float)(1.0 / sqrt((double)ps[v * N + (u < 0 ? u + N : u)])) : 1.0f;
}

// Pass B's results to their slots of D (slot_value_uv's scales).  MX: each bin
// is multiplied by its sqrt w, which also goes to its slot of sqw.
template <bool MX>
__device__ __forceinline__ void dft_store_d(int N, const DftDims& g, const SlotPlan& sp, const int* rows, float2* D,
                                            int rb, int cb, bool pair, const f32x4* dr, const f32x4* di,
                                            const float* __restrict__ ps, float* sqw) {
  const int lane = lane_id(), li = lane & 15, lk = lane >> 4;
  const int hc = pair_cols(N) - 1;
  // this lane's frequency: the pair of columns +-f, or (merged block) f or -f
  const int f = pair ? 16 * cb + li : 16 * (g.nrb - 1) + (li & 7);
  const bool neg = !pair && li >= 8;
  if (f > g.h) return;
  const int4 r4 = *reinterpret_cast<const int4*>(rows + rb * 16 + 4 * lk);
  const int rs[4] = {r4.x, r4.y, r4.z, r4.w};
  const float fs = f == 0 ? 0.70710678118654752f : 1.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = rb * 16 + 4 * lk + j;
    if (r > g.h) continue;
    const float2 a = make_float2(dr[0][j], di[0][j]);
    if (r <= hc && f <= hc) {
      const float sc = (r == 0 ? 0.70710678118654752f : 1.0f) * fs;
      const int at = rs[j] + f;
      float2 z = make_float2(sc * a.x, sc * a.y);
      if (pair) {
        // column 0 is stored as two half-weight copies
        float2 m = f == 0 ? z : make_float2(sc * dr[1][j], sc * di[1][j]);
        if (MX) {
          const float wp = sqrt_weight(ps, N, f, r), wm = sqrt_weight(ps, N, -f, r);
          z = make_float2(z.x * wp, z.y * wp);
          m = make_float2(m.x * wm, m.y * wm);
          *reinterpret_cast<float2*>(sqw + 2 * at) = make_float2(wp, wm);
        }
        *reinterpret_cast<float4*>(D + 2 * at) = make_float4(z.x, z.y, m.x, m.y);
      } else if (f > 0 || !neg) {
        const int v = 2 * at + (neg ? 1 : 0);
        const float w = MX ? sqrt_weight(ps, N, neg ? -f : f, r) : 1.0f;
        if (MX) {
          z = make_float2(z.x * w, z.y * w);
          sqw[v] = w;
          if (f == 0) sqw[v + 1] = w;
        }
        D[v] = z;
        if (f == 0) D[v + 1] = z;
      }
    } else if (!neg) {
      // even N: a Nyquist bin (nyq_bin_uv's order; the last row and frequency
      // are at -h, the mirrors u < 0 of row -h are not stored)
      const bool row = r == g.h, col = f == g.h;
      const int at = 2 * sp.nslots + (row ? (col ? g.h + 1 : f == 0 ? 1 : f + 1) : r == 0 ? 0 : r + g.h + 1);
      const float w = MX ? sqrt_weight(ps, N, f, r) : 1.0f;
      if (MX) sqw[at] = w;
      D[at] = MX ? make_float2(a.x * w, a.y * w) : a;
    }
  }
}

// The whole transform by the workgroup's waves, in region R: the stamp (loaded,
// synchronised) -> D.  tab: the table, in LDS or global memory.  The caller
// synchronises before it reads D (and sqw).
template <int U, bool MX>
__device__ __forceinline__ void stamp_dft(int N, const SlotPlan& sp, const float2* tab, float* R, const int* rows,
                                          const float* __restrict__ ps, float* sqw) {
  const DftDims g = dft_dims(N);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), nw = blockDim.x / kWave;
  f32x4 re[U][2], im[U][2];
  const int ng = (g.nrb + 1) / 2, na = ng * g.ncb;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = wave + u * nw, rb = 2 * (i / g.ncb), cb = i % g.ncb;
    if (i >= na) break;
    if (rb + 1 < g.nrb) dft_pass_a<2>(N, g, R, tab, rb, cb, re[u], im[u]);
    else dft_pass_a<1>(N, g, R, tab, rb, cb, re[u], im[u]);
  }
  __syncthreads();
  float2* Q = reinterpret_cast<float2*>(R);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = wave + u * nw, rb = 2 * (i / g.ncb), cb = i % g.ncb;
    if (i >= na) break;
    dft_store_q(N, g, Q, rb, cb, re[u][0], im[u][0]);
    if (rb + 1 < g.nrb) dft_store_q(N, g, Q, rb + 1, cb, re[u][1], im[u][1]);
  }
  __syncthreads();
  // table blocks of +-u pairs first, then the merged block's half units
  const int npair = g.nblk > g.nrb ? g.nrb - 1 : g.nrb, nb = g.nrb * (npair + g.nblk - g.nrb);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = wave + u * nw, rb = i % g.nrb, cb = i / g.nrb;
    if (i >= nb) break;
    if (cb < npair) dft_pass_b<true>(g, Q, tab, rb, cb, re[u], im[u]);
    else dft_pass_b<false>(g, Q, tab, rb, g.nrb, re[u], im[u]);
  }
  __syncthreads();
  float2* D = reinterpret_cast<float2*>(R);
  const int npc = pair_cols(N);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = wave + u * nw;
    if (i < nb) dft_store_d<MX>(N, g, sp, rows, D, i % g.nrb, i / g.nrb, i / g.nrb < npair, re[u], im[u], ps, sqw);
  }
  for (int sr = wave; sr < sp.nsr; sr += nw)          // padding slots
    for (int s = min(sp.R, npc - sr * sp.R) * npc + lane_id(); s < sp.P * 64; s += kWave) {
      const int t = sr * sp.P * 64 + s;
      D[2 * t] = D[2 * t + 1] = make_float2(0.f, 0.f);
      if (MX) sqw[2 * t] = sqw[2 * t + 1] = 0.f;
    }
  for (int t = 2 * sp.nslots + sp.nspec + threadIdx.x; t < sp.nbins; t += blockDim.x) {
    D[t] = make_float2(0.f, 0.f);
    if (MX) sqw[t] = 0.f;
  }
}

// Waves per workgroup (one stamp at a time) of the transform: one unit each up
// to 8 waves (10,000 stamps of 53 px 172 us so, 275 with two waves of two units
// each, the rest as it was then).
inline int dft_waves(int N) {
  int w = 1;
  while (w < 8 && w < dft_units(N)) w *= 2;
  return w;
}

// Workgroups of a launch over n stamps: as many as are resident with this LDS
// (allocated in pieces of 1,280 bytes) and these waves per SIMD, each taking
// stamp after stamp.
inline int dft_grid(int n, int waves, size_t lds, int per_simd) {
  const int fit = (int)(160 * 1024 / ((lds + 64 + 1279) / 1280 * 1280));
  return std::min(n, 256 * std::max(1, std::min(fit, 4 * per_simd / waves)));
}

}  // namespace bsi
