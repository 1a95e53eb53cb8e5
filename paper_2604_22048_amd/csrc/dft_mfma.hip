// The stamp transforms as dense DFT products on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32, tiles of 16 x 16 accumulated over K steps of 4,
// sizes padded with zeros), one workgroup of 4 waves per galaxy, operands in
// LDS, DFT factors from a 2N-entry twiddle table indexed by the exactly
// reduced phase (pixel centres at x' = x - (N-1)/2).
//
// render_mfma_kernel -- the model stamp (Section 3.2's forward model) from
// the half-plane spectrum T (Hermitian mirror weight 2 on v > 0, the even-N
// Nyquist points weighted as in the float64 renderer):
//   pass 1  B[v][x] = sum_u T[v][u] e^{+i k_u x'}      (rows v = 0..h)
//   pass 2  m[y][x] = N^-2 sum_v Re(B[v][x] e^{+i k_v y'})
// The spectrum's separable factors (PSF, pixel sinc, centroid phase, flux,
// weights) are formed in float64 and rounded; G(q) and the products are
// float32.
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

struct RenderDims {
  int h, ntab, nrow;   // frequency points per row (u = -h..h), rows (v = 0..h)
  int ldT;             // row stride of T: ntab rounded up to 4
  int nrow4;           // rows of B: nrow rounded up to 4
  int Np;              // N rounded up to 16
};

__host__ __device__ inline RenderDims render_dims(int N) {
  RenderDims d;
  d.h = N / 2;
  d.ntab = 2 * d.h + 1;
  d.nrow = d.h + 1;
  d.ldT = (d.ntab + 3) & ~3;
  d.nrow4 = (d.nrow + 3) & ~3;
  d.Np = (N + 15) & ~15;
  return d;
}

// LDS: twiddles [2N], X [ntab], Y [nrow], T [nrow][ldT], B [nrow4][Np] (float2).
__host__ __device__ inline size_t render_mfma_lds(int N) {
  const RenderDims d = render_dims(N);
  return sizeof(float2) * ((size_t)2 * N + d.ntab + d.nrow + (size_t)d.nrow * d.ldT +
                           (size_t)d.nrow4 * d.Np);
}

__global__ void __launch_bounds__(256) render_mfma_kernel(
    const float* __restrict__ params, const float* __restrict__ psf_fwhm, const int32_t* __restrict__ gidx,
    const int64_t* __restrict__ off, int N, float rscale, float pscale_inv, int prof, float nu,
    int n_exp, float* __restrict__ out) {
  extern __shared__ float2 smr[];
  const RenderDims d = render_dims(N);
  const int h = d.h, ntab = d.ntab, nrow = d.nrow, ldT = d.ldT, nrow4 = d.nrow4, Np = d.Np;
  float2* tw = smr;                 // exp(-i pi m / N)
  float2* X = tw + 2 * N;           // u-factor incl. flux and Nyquist weight
  float2* Y = X + ntab;             // v-factor incl. mirror weight
  float2* T = Y + nrow;             // spectrum [nrow][ldT]
  float2* B = T + nrow * ldT;       // half-transform [nrow4][Np]
  const int gal = gidx[blockIdx.x];
  const float* p = params + 6 * (int64_t)(gal / n_exp);     // stamps gal n_exp + j share a galaxy
  const double F = p[0], rpx = (double)p[1] * (double)rscale;
  const float e1 = p[2], e2 = p[3];
  const double dx = p[4], dy = p[5];
  const double sp = (double)psf_fwhm[gal] * 0.42466090014400953 * (double)pscale_inv;
  const bool even = (N & 1) == 0;
  const double kst = 2.0 * 3.14159265358979323846 / (double)N;
  for (int m = threadIdx.x; m < 2 * N; m += blockDim.x) {
    double s, c;
    sincospi((double)m / (double)N, &s, &c);
    tw[m] = make_float2((float)c, (float)(-s));
  }
  for (int t = threadIdx.x; t < ntab + nrow; t += blockDim.x) {
    const bool isx = t < ntab;
    const int f = isx ? t - h : t - ntab;                // u or v
    const double k = f * kst;
    double a = exp(-0.5 * sp * sp * k * k);
    if (f != 0) a *= sinpi((double)f / N) / (3.14159265358979323846 * f / N);
    double s, c;
    sincospi(2.0 * (double)f * (isx ? dx : dy) / (double)N, &s, &c);
    if (isx) {
      a *= F * ((even && (f == h || f == -h)) ? 0.5 : 1.0);
      X[t] = make_float2((float)(a * c), (float)(-a * s));
    } else {
      a *= (f == 0 || (even && f == h)) ? 1.0 : 2.0;
      Y[f] = make_float2((float)(a * c), (float)(-a * s));
    }
  }
  __syncthreads();
  // spectrum T[v][u] = G(q) X(u) Y(v), zero in the padding columns
  {
    const float E = e1 * e1 + e2 * e2;
    const float inv1mE = 1.0f / (1.0f - E);
    const float ca = (1.0f + E + 2.0f * e1) * inv1mE, cb = (1.0f + E - 2.0f * e1) * inv1mE;
    const float cc = 4.0f * e2 * inv1mE;
    const float r2 = (float)(rpx * rpx), ks = (float)kst;
    for (int t = threadIdx.x; t < nrow * ldT; t += blockDim.x) {
      const int v = t / ldT, c = t - v * ldT;
      float2 z = make_float2(0.f, 0.f);
      if (c < ntab) {
        const float kx = (float)(c - h) * ks, ky = (float)v * ks;
        const float q = fmaf(ca, kx * kx, fmaf(cb, ky * ky, cc * kx * ky));
        float G;
        if (prof == kProfExp) {
          const float rs = rsqrtf(fmaf(r2, q, 1.0f));
          G = rs * rs * rs;
        } else if (prof == kProfSpergel) {
          G = exp2f(-(1.0f + nu) * log2f(fmaf(r2, q, 1.0f)));
        } else {
          G = expf(-0.5f * r2 * q);
        }
        const float2 x = X[c], y = Y[v];
        z = make_float2(G * fmaf(x.x, y.x, -x.y * y.y), G * fmaf(x.x, y.y, x.y * y.x));
      }
      T[t] = z;
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;      // operand row/column, K index within a step
  // pass 1: tiles of B (16 rows v x 16 columns x), Re and Im accumulated together
  const int nrb = (nrow + 15) >> 4, ncb = Np >> 4;
  for (int ti = wave; ti < nrb * ncb; ti += 4) {
    const int rb = ti / ncb, cb = ti - rb * ncb;
    const int v = rb * 16 + li, x = cb * 16 + li;
    // twiddle index of (u = k - h, x), advanced by 4 in u per step
    int m = tw_index(lk - h, x, N);
    const int st4 = tw_index(4, x, N);
    f32x4 br = {0.f, 0.f, 0.f, 0.f}, bi = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < ldT; k0 += 4) {
      const int k = k0 + lk;
      const float2 a = (v < nrow) ? T[v * ldT + k] : make_float2(0.f, 0.f);
      float C = 0.f, S = 0.f;
      if (k < ntab && x < N) {
        const float2 w = tw[m];                        // exp(-i k_u x'); e^{+i..} = conj
        C = w.x;
        S = -w.y;
      }
      m += st4;
      if (m >= 2 * N) m -= 2 * N;
      br = mfma16x16x4(a.x, C, br);
      br = mfma16x16x4(-a.y, S, br);
      bi = mfma16x16x4(a.x, S, bi);
      bi = mfma16x16x4(a.y, C, bi);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rb * 16 + 4 * lk + r;
      if (row < nrow4) B[row * Np + x] = make_float2(br[r], bi[r]);
    }
  }
  __syncthreads();
  // pass 2: tiles of m (16 rows y x 16 columns x), K = v
  const float inv = (float)(1.0 / ((double)N * (double)N));
  const int64_t o = off[gal];
  const int nb = Np >> 4;
  for (int ti = wave; ti < nb * nb; ti += 4) {
    const int yb = ti / nb, xb = ti - yb * nb;
    const int y = yb * 16 + li, x = xb * 16 + li;
    int m = tw_index(lk, y, N);                        // (v, y), advanced by 4 in v per step
    const int st4 = tw_index(4, y, N);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nrow4; k0 += 4) {
      const int v = k0 + lk;
      float cy = 0.f, sy = 0.f;
      float2 b = make_float2(0.f, 0.f);
      if (v < nrow) {
        if (y < N) {
          const float2 w = tw[m];                      // Re(b e^{+i k_v y'}) = b.x w.x + b.y w.y
          cy = w.x;
          sy = w.y;
        }
        b = B[v * Np + x];
      }
      m += st4;
      if (m >= 2 * N) m -= 2 * N;
      acc = mfma16x16x4(cy, b.x, acc);
      acc = mfma16x16x4(sy, b.y, acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int yy = yb * 16 + 4 * lk + r;
      if (yy < N && x < N) out[o + (int64_t)yy * N + x] = acc[r] * inv;
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
  if (!BIG) load_table(N, tab, t);
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

size_t render_mfma_lds_bytes(int N) { return render_mfma_lds(N); }
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
  e = hipGetLastError();
  const hipError_t e2 = hipStreamSynchronize(s);
  (void)hipStreamDestroy(s);
  if (e == hipSuccess) e = e2;
  done[device] = e == hipSuccess;
  return e;
}

DftTab dft_tables(int N) {
  static std::mutex m;
  static void* ptr[kMaxDevices][2] = {};
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return {nullptr, nullptr};
  std::lock_guard<std::mutex> lock(m);
  void** p = ptr[device];
  if (!p[1]) {
    if (hipGetSymbolAddress(&p[0], HIP_SYMBOL(dft_tab)) != hipSuccess) return {nullptr, nullptr};
    if (hipGetSymbolAddress(&p[1], HIP_SYMBOL(sinc_tab)) != hipSuccess) return {nullptr, nullptr};
  }
  static const auto offs = [] {
    std::array<int, kMaxN + 1> o{};
    for (int n = 8; n < kMaxN; ++n) o[n + 1] = o[n] + dft_tab_len(n);
    return o;
  }();
  return {static_cast<const float2*>(p[0]) + offs[N], static_cast<const double2*>(p[1]) + N * kSincLen};
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

hipError_t launch_render_mfma(const float* params, const float* psf, const int32_t* gidx, int n,
                              const int64_t* off, int N, float rscale, float pscale_inv, int prof, float nu,
                              float* out, hipStream_t s, int n_exp) {
  if (n <= 0) return hipSuccess;
  const size_t lds = render_mfma_lds(N);
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  (void)hipFuncSetAttribute((const void*)render_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
  hipLaunchKernelGGL(render_mfma_kernel, dim3(n), dim3(256), lds, s, params, psf, gidx, off, N, rscale,
                     pscale_inv, prof, nu, n_exp, out);
  return hipGetLastError();
}

}  // namespace bsi
