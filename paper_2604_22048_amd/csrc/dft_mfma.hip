// The stamp transforms as dense DFT products on the matrix cores (tiles of 16 x
// 16 accumulated over K steps of 4, sizes padded with zeros), a workgroup per
// stamp at a time, operands in LDS, DFT factors from per-device tables laid
// out as the operands are held.
//
// render_mfma_kernel -- the model stamp (Section 3.2's forward model) from
// the half-plane spectrum T (Hermitian mirror weight 2 on v > 0, the even-N
// Nyquist points weighted as in the float64 renderer), folded about the
// stamp's centre: pixels at +-x' and frequencies +-u share cos(k_u x') and
// sin(k_u x'), so with S, D = T(u) +- T(-u) (u >= 0)
//   pass 1  E, O = sum_u S cos(k_u x'), sum_u D sin(k_u x')  (v = 0..h, x' >= 0)
//           B(+-x') = E +- i O,  B[v][x] = sum_u T[v][u] e^{+i k_u x'}
//   pass 2  m(y', +-x') = N^-2 sum_v Re(B e^{+i k_v y'}), likewise from
//           C_E, C_O = sum_v Re E cos, Im O cos and S_E, S_O = sum_v Im E sin,
//           Re O sin: four pixels (+-y', +-x') per element
// a third of the products of the unfolded form.  In float32 (the spectrum's
// separable factors -- PSF, pixel sinc, centroid phase, flux, weights -- formed
// in float64 and rounded) for bsi_render_stamps, in float64 throughout for the
// pixel-space likelihood.
//
// dft_bins_mfma_kernel -- the forward DFT of a stamp (or of data - model) at the
// half-plane bins of the k-space likelihood, written in slot order
// (dft_device.h).
#include <algorithm>
#include <array>
#include <mutex>

#include "bsi_kernels.h"
#include "dft_device.h"

namespace bsi {

namespace {

// ---- tables ------------------------------------------------------------------

constexpr int kDftTabLen = dft_tab_off(kMaxN + 1);
__device__ __align__(16) float2 dft_tab[kDftTabLen + kAhead * 64];       // 4 MB
__device__ double2 sinc_tab[(kMaxN + 1) * kSincLen];

// One block per stamp side from 8: the side's operands and {k_u, sinc} pairs.
__global__ void __launch_bounds__(256) dft_tables_kernel() {
  const int N = 8 + blockIdx.x;
  const DftDims d = dft_dims(N);
  float2* tab = dft_tab + dft_tab_off(N);
  for (int t = threadIdx.x; t < d.nblk * d.steps * 64; t += blockDim.x) {
    const int lane = t & 63, s = (t >> 6) % d.steps, blk = (t >> 6) / d.steps;
    const int li = lane & 15, pix = 4 * s + (lane >> 4);
    const bool merged = blk == d.nrb;
    const int f = merged ? 16 * (d.nrb - 1) + (li & 7) : 16 * blk + li;
    float2 w = make_float2(0.f, 0.f);
    if (pix < N && f <= d.h) {
      const bool neg = (merged && li >= 8) || ((N & 1) == 0 && f == d.h);   // (Nyquist: -h)
      double sn, c;
      sincospi((double)tw_index(neg ? -f : f, pix, N) / (double)N, &sn, &c);
      w = make_float2((float)c, (float)(-sn));
    }
    tab[t] = w;
  }
  for (int u = threadIdx.x; u <= d.h; u += blockDim.x)
    sinc_tab[N * kSincLen + u] =
        make_double2(2.0 * 3.14159265358979323846 * u / N,
                     u == 0 ? 1.0 : sinpi((double)u / N) / (3.14159265358979323846 * u / N));
}

// ---- render ------------------------------------------------------------------

struct RenderDims {
  int h, nrow;         // frequencies 0..h of either axis
  int nh;              // pixel distances x' >= 0 from the centre
  int nrb, ntb;        // 16-blocks of frequencies and of distances
  int steps;           // K steps of 4 frequencies
  int ldS;             // row stride of (S, D): odd, so that 16 rows' reads fall on all banks
};

__host__ __device__ constexpr RenderDims render_dims(int N) {
  RenderDims d{};
  d.h = N / 2;
  d.nrow = d.h + 1;
  d.nh = (N + 1) / 2;
  d.nrb = (d.nrow + 15) / 16;
  d.ntb = (d.nh + 15) / 16;
  d.steps = (d.nrow + 3) / 4;
  d.ldS = 4 * d.steps + 1;
  return d;
}

// Table entries of one side, [ntb][steps][64]: {cos, sin}(k_f x'_t), t = 16 block
// + lane % 16, f = 4 step + lane / 16.
__host__ __device__ constexpr int render_tab_len(int N) {
  const RenderDims d = render_dims(N);
  return d.ntb * d.steps * 64;
}

__host__ __device__ constexpr int render_tab_off(int N) {
  int o = 0;
  for (int n = 8; n < N; ++n) o += render_tab_len(n);
  return o;
}

// The kernel's arithmetic: vectors, the 16 x 16 x 4 product, and the row of
// element e of an accumulator on lane group lk.
template <typename T>
struct Mf;
template <>
struct Mf<float> {
  typedef float4 V4;
  typedef float2 V2;
  typedef f32x4 Acc;
  static __device__ __forceinline__ Acc mul(float a, float b, Acc c) { return mfma16x16x4(a, b, c); }
  static __device__ __forceinline__ int row(int lk, int e) { return 4 * lk + e; }
};
template <>
struct Mf<double> {
  typedef double4 V4;
  typedef double2 V2;
  typedef double Acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ Acc mul(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int e) { return lk + 4 * e; }
};

__device__ __align__(16) float2 render_tab_f[render_tab_off(kMaxN + 1) + 64];
__device__ __align__(16) double2 render_tab_d[render_tab_off(kMaxN + 1)];

__global__ void __launch_bounds__(256) render_tables_kernel() {
  const int N = 8 + blockIdx.x;
  const RenderDims d = render_dims(N);
  const int o = render_tab_off(N);
  for (int e = threadIdx.x; e < d.ntb * d.steps * 64; e += blockDim.x) {
    const int lane = e & 63, t = (e >> 6) / d.steps * 16 + (lane & 15), f = (e >> 6) % d.steps * 4 + (lane >> 4);
    double2 w = make_double2(0.0, 0.0);
    if (t < d.nh && f <= d.h) {
      // k_f x' = pi f (2 x') / N, 2 x' = 2 t (odd N) or 2 t + 1
      const int m = f * (2 * t + (N & 1 ? 0 : 1)) % (2 * N);
      sincospi((double)m / (double)N, &w.y, &w.x);
    }
    render_tab_d[o + e] = w;
    render_tab_f[o + e] = make_float2((float)w.x, (float)w.y);
  }
}

// LDS: (S, D) [nrow][ldS] and then (E, O) [4 steps][16 ntb] in one region, the
// table (float32 only), X [h + 1], Y [h + 1].
template <typename T>
struct RenderLds {
  size_t tab, xy, total;
};

template <typename T>
__host__ __device__ inline RenderLds<T> render_lds(int N) {
  const RenderDims d = render_dims(N);
  const size_t a = sizeof(T) * 4 * (size_t)d.nrow * d.ldS, b = sizeof(T) * 4 * (size_t)d.steps * 4 * d.ntb * 16;
  RenderLds<T> l;
  l.tab = a > b ? a : b;
  l.xy = l.tab + (sizeof(T) == 4 ? sizeof(T) * 2 * ((size_t)d.ntb * d.steps * 64 + 64) : 0);
  l.total = l.xy + sizeof(T) * 4 * (size_t)d.nrow;
  return l;
}

__host__ __device__ constexpr int render_units(int N) {
  const RenderDims d = render_dims(N);
  return d.nrb > d.ntb ? d.nrb * d.ntb : d.ntb * d.ntb;
}

// Profile factor G(q), r the profile's scale in pixels.
__device__ __forceinline__ float profile_g(int prof, float nu, float r2, float q) {
  if (prof == kProfExp) {
    const float rs = rsqrtf(fmaf(r2, q, 1.0f));
    return rs * rs * rs;
  }
  if (prof == kProfSpergel) return exp2f(-(1.0f + nu) * log2f(fmaf(r2, q, 1.0f)));
  return expf(-0.5f * r2 * q);
}

__device__ __forceinline__ double profile_g(int prof, float nu, double r2, double q) {
  if (prof == kProfExp) {
    const double a = 1.0 + r2 * q;
    return 1.0 / (a * sqrt(a));
  }
  if (prof == kProfSpergel) return pow(1.0 + r2 * q, -(1.0 + (double)nu));
  return exp(-0.5 * r2 * q);
}

// U units (16 x 16 blocks of four sums) per wave and pass.  Bound by the
// latencies between its barriers, the matrix cores and the spectrum's
// arithmetic about equally.  float32, 10,000 stamps of 53 px 125 us a call (262
// unfolded, with the factors looked up and their table built per stamp), 1,000
// of 101 px 65 us (284); float64 with the likelihood, 1,000 of 41 px 57 us, one
// of 101 px 74 us (direct float64 sums, a row of the spectrum at a time: 291, 822).
// The float64 form of three units (the largest sides) spills 72 of its 256
// registers, the most that a workgroup of eight waves can have.
template <typename T, int U>
__global__ void __launch_bounds__(512, sizeof(T) == 4 && U == 1 ? 4 : 2) render_mfma_kernel(
    const float* __restrict__ params, const float* __restrict__ psf_fwhm, const int32_t* __restrict__ gidx, int n,
    const int64_t* __restrict__ off, int N, float rscale, float pscale_inv, int prof, float nu, int n_exp,
    const void* __restrict__ tabv, const double2* __restrict__ sinc, T* __restrict__ out) {
  typedef typename Mf<T>::V4 V4;
  typedef typename Mf<T>::V2 V2;
  typedef typename Mf<T>::Acc Acc;
  extern __shared__ float4 smr4[];
  const RenderDims d = render_dims(N);
  const RenderLds<T> l = render_lds<T>(N);
  char* base = reinterpret_cast<char*>(smr4);
  V4* SD = reinterpret_cast<V4*>(base);
  V4* EO = SD;
  V2* X = reinterpret_cast<V2*>(base + l.xy);      // u-factor incl. flux and Nyquist weight
  V2* Y = X + d.nrow;                              // v-factor incl. mirror weight
  const V2* tab = static_cast<const V2*>(tabv);
  const V2* tb = tab;
  if constexpr (sizeof(T) == 4) {
    V2* t = reinterpret_cast<V2*>(base + l.tab);
    load_table(tab, t, render_tab_len(N));
    wait_loads();
    tb = t;
  }
  const bool even = (N & 1) == 0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), nw = blockDim.x / kWave;
  const int lane = lane_id(), li = lane & 15, lk = lane >> 4;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const int gal = gidx ? gidx[i] : i;
    const float* p = params + 6 * (int64_t)(gal / n_exp);     // stamps gal n_exp + j share a galaxy
    const double F = p[0], rpx = (double)p[1] * (double)rscale;
    const double sp = (double)psf_fwhm[gal] * 0.42466090014400953 * (double)pscale_inv;
    for (int t = threadIdx.x; t < 2 * d.nrow; t += blockDim.x) {
      const bool isx = t < d.nrow;
      const int f = isx ? t : t - d.nrow;
      const double2 ks = sinc[f];
      double a = exp(-0.5 * sp * sp * ks.x * ks.x) * ks.y;
      double s, c;
      sincospi(2.0 * (double)f * (double)p[isx ? 4 : 5] / (double)N, &s, &c);
      a *= isx ? F * (even && f == d.h ? 0.5 : 1.0) : (f == 0 || (even && f == d.h)) ? 1.0 : 2.0;
      V2 z;
      z.x = (T)(a * c);
      z.y = (T)(-a * s);
      X[t] = z;
    }
    __syncthreads();
    // T(+-u, v) = G X(+-u) Y(v), X(-u) = conj X(u): sums and differences, zero
    // in the padding columns
    {
      const T e1 = p[2], e2 = p[3];
      const T E = e1 * e1 + e2 * e2, inv1mE = (T)1 / ((T)1 - E);
      const T ca = ((T)1 + E + (T)2 * e1) * inv1mE, cb = ((T)1 + E - (T)2 * e1) * inv1mE;
      const T cc = (T)4 * e2 * inv1mE, r2 = (T)(rpx * rpx), kst = (T)(2.0 * 3.14159265358979323846 / (double)N);
      for (int t = threadIdx.x; t < d.nrow * 4 * d.steps; t += blockDim.x) {
        const int v = t / (4 * d.steps), u = t - v * 4 * d.steps;
        V4 z;
        z.x = z.y = z.z = z.w = (T)0;
        if (u <= d.h) {
          const T kx = (T)u * kst, ky = (T)v * kst;
          const T qa = fma(ca, kx * kx, cb * ky * ky), qc = cc * kx * ky;
          const V2 x = X[u], y = Y[v];
          const T a = x.y * y.y, b = x.y * y.x;
          const T Gp = profile_g(prof, nu, r2, qa + qc);
          const T pr = Gp * fma(x.x, y.x, -a), pi = Gp * fma(x.x, y.y, b);
          if (u == 0) {
            z.x = pr;
            z.y = pi;
          } else {
            const T Gm = profile_g(prof, nu, r2, qa - qc);
            const T mr = Gm * fma(x.x, y.x, a), mi = Gm * fma(x.x, y.y, -b);
            z.x = pr + mr;
            z.y = pi + mi;
            z.z = pr - mr;
            z.w = pi - mi;
          }
        }
        SD[v * d.ldS + u] = z;
      }
    }
    __syncthreads();
    Acc acc[U][4];
    // pass 1: E, O (Re, Im) at 16 frequencies v x 16 distances x'
#pragma unroll
    for (int w = 0; w < U; ++w) {
      const int k = wave + w * nw, rb = k / d.ntb, cb = k % d.ntb;
      if (rb >= d.nrb) break;
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[w][q] = Acc{0, 0, 0, 0};
      const V4* ap = SD + min(rb * 16 + li, d.nrow - 1) * d.ldS + lk;
      const V2* bp = tb + cb * d.steps * 64 + lane;
#pragma unroll 2
      for (int s = 0; s < d.steps; ++s) {
        const V4 a = ap[4 * s];
        const V2 b = bp[s * 64];
        acc[w][0] = Mf<T>::mul(a.x, b.x, acc[w][0]);
        acc[w][1] = Mf<T>::mul(a.y, b.x, acc[w][1]);
        acc[w][2] = Mf<T>::mul(a.z, b.y, acc[w][2]);
        acc[w][3] = Mf<T>::mul(a.w, b.y, acc[w][3]);
      }
    }
    __syncthreads();
    const int ldE = 16 * d.ntb;
#pragma unroll
    for (int w = 0; w < U; ++w) {
      const int k = wave + w * nw, rb = k / d.ntb, cb = k % d.ntb;
      if (rb >= d.nrb) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = rb * 16 + Mf<T>::row(lk, e);
        V4 z;
        z.x = acc[w][0][e];
        z.y = acc[w][1][e];
        z.z = acc[w][2][e];
        z.w = acc[w][3][e];
        if (v >= d.nrow) z.x = z.y = z.z = z.w = (T)0;       // up to a whole K step
        if (v < 4 * d.steps) EO[v * ldE + cb * 16 + li] = z;
      }
    }
    __syncthreads();
    // pass 2: C_E, C_O, S_E, S_O at 16 distances y' x 16 distances x'
#pragma unroll
    for (int w = 0; w < U; ++w) {
      const int k = wave + w * nw, yb = k / d.ntb, xb = k % d.ntb;
      if (yb >= d.ntb) break;
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[w][q] = Acc{0, 0, 0, 0};
      const V2* ap = tb + yb * d.steps * 64 + lane;
      const V4* bp = EO + lk * ldE + xb * 16 + li;
#pragma unroll 2
      for (int s = 0; s < d.steps; ++s) {
        const V2 a = ap[s * 64];
        const V4 b = bp[4 * s * ldE];
        acc[w][0] = Mf<T>::mul(a.x, b.x, acc[w][0]);
        acc[w][1] = Mf<T>::mul(a.x, b.w, acc[w][1]);
        acc[w][2] = Mf<T>::mul(a.y, b.y, acc[w][2]);
        acc[w][3] = Mf<T>::mul(a.y, b.z, acc[w][3]);
      }
    }
    __syncthreads();        // the region is free for the next stamp
    const T inv = (T)(1.0 / ((double)N * (double)N));
    T* o = out + (off ? off[gal] : (int64_t)gal * N * N);
#pragma unroll
    for (int w = 0; w < U; ++w) {
      const int k = wave + w * nw, yb = k / d.ntb, xb = k % d.ntb;
      if (yb >= d.ntb) break;
      const int tx = xb * 16 + li;
      if (tx >= d.nh) continue;
      const int xp = d.h + tx, xm = d.h - tx - (even ? 1 : 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ty = yb * 16 + Mf<T>::row(lk, e);
        if (ty >= d.nh) continue;
        const T cp = acc[w][0][e] - acc[w][1][e], cm = acc[w][0][e] + acc[w][1][e];
        const T sp2 = acc[w][2][e] + acc[w][3][e], sm = acc[w][2][e] - acc[w][3][e];
        // (on the centre row and column of an odd N both signs name one pixel)
        T* rp = o + (int64_t)(d.h + ty) * N;
        T* rm = o + (int64_t)(d.h - ty - (even ? 1 : 0)) * N;
        rp[xp] = (cp - sp2) * inv;
        if (xm != xp) rp[xm] = (cm - sm) * inv;
        if (rm != rp) {
          rm[xp] = (cp + sp2) * inv;
          if (xm != xp) rm[xm] = (cm + sm) * inv;
        }
      }
    }
  }
}

// U units per wave (dft_per_wave); with four (dft_big) the DFT table is read from
// memory instead of LDS.  Bound by the matrix cores, 55 % busy: the stamp's way
// in and the spectrum's way out are under other workgroups' products (5 per
// compute unit at 53 px).  10,000 stamps of 53 px: 150 us (218 with the factors
// from a 2N-entry table, one stamp per workgroup).
template <int U>
__global__ void __launch_bounds__(512, U == 1 ? 5 : U == 2 ? 4 : 2) dft_bins_mfma_kernel(
    const float* __restrict__ data, const double* __restrict__ model, const int32_t* __restrict__ gidx, int n,
    const int64_t* __restrict__ off, const int64_t* __restrict__ bin_off, int N, int P,
    const float2* __restrict__ tab, float2* __restrict__ out, double* __restrict__ chi2) {
  constexpr bool BIG = U > 2;
  extern __shared__ float4 smd4[];
  __shared__ double red[8];
  const SlotPlan sp = make_slot_plan_p(N, P);
  const DftLds l = dft_lds(N, sp);
  char* base = reinterpret_cast<char*>(smd4);
  float* R = reinterpret_cast<float*>(base);
  int* rows = reinterpret_cast<int*>(base + l.r);
  float2* t = reinterpret_cast<float2*>(base + l.r + l.rows);
  if (!BIG) load_table(tab, t, dft_tab_len(N));
  dft_row_bases(N, sp, rows);
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const int gal = gidx[i];
    const int64_t o = off[gal];
    double sq = load_stamp(N, data + o, model ? model + o : nullptr, R);
    if (chi2) {
      sq = wave_sum(sq);
      if (lane_id() == 0) red[threadIdx.x / kWave] = sq;
    }
    __syncthreads();
    if (chi2 && threadIdx.x == 0) {
      double tot = 0.0;
      for (int w = 0; w < (int)(blockDim.x / kWave); ++w) tot += red[w];
      chi2[gal] = tot;
    }
    const float next = i + gridDim.x < n ? touch_stamp(N, data + off[gidx[i + gridDim.x]]) : 0.f;
    stamp_dft<U, false>(N, sp, BIG ? tab : t, R, rows, nullptr, nullptr);
    touch_done(next);
    __syncthreads();
    // nbins is even, and so is every spectrum's offset
    float4* dst = reinterpret_cast<float4*>(out + bin_off[gal]);
    const float4* src = reinterpret_cast<const float4*>(R);
    for (int b = threadIdx.x; b < sp.nbins / 2; b += blockDim.x) dst[b] = src[b];
    __syncthreads();
  }
}

constexpr size_t kMaxDftLds = 160 * 1024 - 64;     // beside the static scratch

}  // namespace

hipError_t init_dft_tables(int device) {
  static std::mutex m;
  static bool done[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(m);
  if (done[device]) return hipSuccess;
  hipStream_t s = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(dft_tables_kernel, dim3(kMaxN - 7), dim3(256), 0, s);
  hipLaunchKernelGGL(render_tables_kernel, dim3(kMaxN - 7), dim3(256), 0, s);
  e = hipGetLastError();
  const hipError_t e2 = hipStreamSynchronize(s);
  (void)hipStreamDestroy(s);
  if (e == hipSuccess) e = e2;
  done[device] = e == hipSuccess;
  return e;
}

namespace {

// Addresses of the current device's tables (NULL if they cannot be read).
struct TabPtrs {
  void *dft, *sinc, *render_f, *render_d;
};

TabPtrs table_ptrs() {
  static std::mutex m;
  static TabPtrs ptr[kMaxDevices] = {};
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return {};
  std::lock_guard<std::mutex> lock(m);
  TabPtrs& p = ptr[device];
  if (!p.render_d) {
    TabPtrs q{};
    if (hipGetSymbolAddress(&q.dft, HIP_SYMBOL(dft_tab)) != hipSuccess ||
        hipGetSymbolAddress(&q.sinc, HIP_SYMBOL(sinc_tab)) != hipSuccess ||
        hipGetSymbolAddress(&q.render_f, HIP_SYMBOL(render_tab_f)) != hipSuccess ||
        hipGetSymbolAddress(&q.render_d, HIP_SYMBOL(render_tab_d)) != hipSuccess)
      return {};
    p = q;
  }
  return p;
}

template <int (*LEN)(int)>
int table_off(int N) {
  static const auto offs = [] {
    std::array<int, kMaxN + 1> o{};
    for (int n = 8; n < kMaxN; ++n) o[n + 1] = o[n] + LEN(n);
    return o;
  }();
  return offs[N];
}

}  // namespace

DftTab dft_tables(int N) {
  const TabPtrs p = table_ptrs();
  if (!p.dft) return {nullptr, nullptr};
  return {static_cast<const float2*>(p.dft) + table_off<dft_tab_len>(N),
          static_cast<const double2*>(p.sinc) + N * kSincLen};
}

size_t dft_bins_mfma_lds_bytes(int N, int P) {
  const DftLds l = dft_lds(N, make_slot_plan_p(N, P));
  return l.r + l.rows + (dft_big(N) ? 0 : l.tab);
}

hipError_t launch_dft_bins_mfma(const float* data, const double* model, const int32_t* gidx, int n,
                                const int64_t* off, const int64_t* bin_off, int N, int P, float2* out,
                                double* chi2, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const size_t lds = dft_bins_mfma_lds_bytes(N, P);
  const DftTab t = dft_tables(N);
  if (lds > kMaxDftLds || !t.dft) return hipErrorInvalidValue;
  const int per = dft_per_wave(N);
  auto kern = per == 1 ? dft_bins_mfma_kernel<1> : per == 2 ? dft_bins_mfma_kernel<2> : dft_bins_mfma_kernel<4>;
  const int nw = dft_waves(N);
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(dft_grid(n, nw, lds, per == 1 ? 5 : per == 2 ? 4 : 2)), dim3(kWave * nw), lds, s, data, model, gidx, n, off, bin_off,
                     N, P, t.dft, out, chi2);
  return hipGetLastError();
}

template <typename T>
static hipError_t render_impl(const float* params, const float* psf, const int32_t* gidx, int n, const int64_t* off,
                              int N, float rscale, float pscale_inv, int prof, float nu, T* out, hipStream_t s,
                              int n_exp) {
  if (n <= 0) return hipSuccess;
  const size_t lds = render_lds<T>(N).total;
  const TabPtrs t = table_ptrs();
  if (lds > 160 * 1024 || !t.sinc) return hipErrorInvalidValue;
  const auto* tab = static_cast<const typename Mf<T>::V2*>(sizeof(T) == 4 ? t.render_f : t.render_d) +
                    table_off<render_tab_len>(N);
  int nw = 1;
  while (nw < 8 && nw < render_units(N)) nw *= 2;
  auto go = [&](auto kern, int per_simd) {
    if (lds > 64 * 1024)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(dft_grid(n, nw, lds, per_simd)), dim3(kWave * nw), lds, s, params, psf, gidx, n, off,
                       N, rscale, pscale_inv, prof, nu, n_exp, static_cast<const void*>(tab),
                       static_cast<const double2*>(t.sinc) + N * kSincLen, out);
  };
  // units per wave: one up to 8, two up to 16, three (20 at most: 128 px)
  if (render_units(N) <= 8) go(render_mfma_kernel<T, 1>, sizeof(T) == 4 ? 4 : 2);
  else if (render_units(N) <= 16) go(render_mfma_kernel<T, 2>, 2);
  else go(render_mfma_kernel<T, 3>, 2);
  return hipGetLastError();
}

hipError_t launch_render_mfma(const float* params, const float* psf, const int32_t* gidx, int n, const int64_t* off,
                              int N, float rscale, float pscale_inv, int prof, float nu, float* out, hipStream_t s,
                              int n_exp) {
  return render_impl(params, psf, gidx, n, off, N, rscale, pscale_inv, prof, nu, out, s, n_exp);
}

hipError_t launch_render_f64(const float* params, const float* psf, const int32_t* gidx, int n, const int64_t* off,
                             int N, float rscale, float pscale_inv, int prof, float nu, double* out, hipStream_t s) {
  return render_impl(params, psf, gidx, n, off, N, rscale, pscale_inv, prof, nu, out, s, 1);
}

}  // namespace bsi
