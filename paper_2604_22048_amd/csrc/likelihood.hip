// Batched log-likelihood and gradient (eq. likelihood-pixels), one workgroup per
// galaxy: the DFT of the stamp (or, for the pixel method, of the pixel
// residual) at the half-plane bins is formed in LDS by all its waves
// (dft_device.h) and contracted there with the analytic spectrum by one of
// them (kspace_sums, the routine the sampler uses), so the spectrum never
// leaves the workgroup.  With the direct transform, which is a kernel of its
// own, the spectra are read from memory instead.
#include <type_traits>

#include "bsi_kernels.h"
#include "dft_device.h"

namespace bsi {

namespace {

constexpr size_t kMaxLds = 160 * 1024 - 128;    // beside the static scratch

// LDS: [stamp, then spectrum | sqrt-weights | column table | PSF-sinc table | row
// bases | Ym, X, Yf | reduction scratch | DFT table]; only the column and
// PSF-sinc tables, Ym, X, Yf and the scratch where the spectra come from memory.
struct LoglikLds {
  size_t sqw, cols, atab, rows, sep, red, tab, total;      // byte offsets
};

__host__ __device__ inline LoglikLds loglik_lds(int N, int P, bool mx, bool fused) {
  const Geom g = make_geom(N);
  const SlotPlan sp = make_slot_plan_p(N, P);
  const DftLds f = dft_lds(N, sp);
  auto up = [](size_t b) { return (b + 15) & ~(size_t)15; };
  LoglikLds l;
  l.sqw = fused ? f.r : 0;
  l.cols = l.sqw + (fused && mx ? up(sizeof(float) * sp.nbins) : 0);
  l.atab = l.cols + sizeof(float4) * sp.P * 64;
  l.rows = l.atab + up(sizeof(float) * g.ntab);
  l.sep = l.rows + (fused ? f.rows : 0);
  l.red = l.sep + sizeof(float4) * sp.ymax + up(sizeof(float2) * (2 * g.ntab + 3));
  l.tab = l.red + sizeof(float) * 64 * 8;
  l.total = l.tab + (fused ? f.tab : 0);
  return l;
}

// Waves per SIMD that a form's registers leave room for.  One unit without
// weights: four, under whose 128 registers the contraction spills 4 to 36 where
// three would take 146 and spill none, but hide less (10,000 stamps of 53 px 185
// against 195 us, 41 px 132 against 143).  With weights, which would spill 46 to 56
// (two units: 89 and more): three (8 to 12 left; 10,000 of 53 px 290 -> 252 us, 700
// of three exposures 70 -> 63).  Two units, whose workgroups of eight waves LDS
// mostly leaves room for one of: three as well, which keeps room for another
// side's four waves beside them (up to 15 left, 38 with weights, where 300 bytes a
// lane were spilled; 700 of 73 px with weights 96 -> 74 us, 700 of 101 px 103 -> 94).
// Two would spill none and take 5 to 15 % less for a side alone with weights (700
// of 73 px 66), but mixed batches up to 15 % more (1,000 galaxies of 32, 48 and
// 64 px, three exposures: 220 against 192).
constexpr int loglik_simd_waves(int P, bool mx, int U) {
  return U == 0 ? 1 : P > 4 ? 2 : U == 2 || mx ? 3 : 4;
}

// MX: the sum over the galaxy's n_exp exposures (stamps gal n_exp + j, each
// transformed in turn) with per-bin noise weights (Appendix C).
// U units of the transform per wave (dft_per_wave), or U = 0: the spectra come
// from memory, one wave per galaxy.
// Bound by the matrix cores (the transform's products, half of the time) and by
// what runs beside them: 4 workgroups of 4 waves per compute unit at 53 px,
// some contracting with one wave while the others transform.  10,000 galaxies
// of 53 px: 185 us a call, calls queued back to back; transform and contraction as two kernels, with
// the transform's factors looked up per element and the spectra (123 MB)
// through memory and LDS, took 218 and 69.
template <int PROF, bool RESID, int P, bool MX, int U>
__global__ void __launch_bounds__(U == 0 ? kWave : 512, loglik_simd_waves(P, MX, U)) loglik_kernel(LoglikArgs a) {
  static_assert(!(MX && RESID), "exposures: k-space form only");
  extern __shared__ float4 smem4[];
  __shared__ double red[8];
  const int N = a.N;
  const Geom g = make_geom(N);
  const SlotPlan sp = make_slot_plan_p(N, P);
  constexpr bool FUSED = U > 0;
  const LoglikLds l = loglik_lds(N, P, MX, FUSED);
  char* base = reinterpret_cast<char*>(smem4);
  float* R = reinterpret_cast<float*>(base);
  float* sqw_s = reinterpret_cast<float*>(base + l.sqw);
  float4* cols = reinterpret_cast<float4*>(base + l.cols);
  float* atab = reinterpret_cast<float*>(base + l.atab);
  int* rows = reinterpret_cast<int*>(base + l.rows);
  float2* tab = reinterpret_cast<float2*>(base + l.tab);
  float4* Ym = reinterpret_cast<float4*>(base + l.sep);
  float2* X = reinterpret_cast<float2*>(Ym + sp.ymax);
  float2* Yf = X + g.ntab + 2;
  float* scratch = reinterpret_cast<float*>(base + l.red);
  if (FUSED) {
    load_table(a.tab.dft, tab, dft_tab_len(N));
    dft_row_bases(N, sp, rows);
  }
  build_col_table(g, sp, cols);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), nw = blockDim.x / kWave;
  const int ne = MX ? a.n_exp : 1;
  for (int gi = blockIdx.x; gi < a.n; gi += gridDim.x) {
    const int gal = a.gidx ? a.gidx[gi] : gi;
    const float* p = a.params + 6 * (int64_t)gal;
    const float F = p[0], s = p[1], e1 = p[2], e2 = p[3], dx = p[4], dy = p[5];
    const float E = e1 * e1 + e2 * e2;
    const Shape sh = make_shape<PROF>(s * a.rscale, e1, e2, a.nu);
    KResult r{0.0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float sig = 1.0f;
    for (int x = 0; x < ne; ++x) {
      const int64_t st = MX ? (int64_t)gal * ne + x : gal;    // this exposure's stamp
      const int64_t o = a.off ? a.off[st] : st * N * N;
      __syncthreads();                                        // the last stamp has been summed
      double sq = 0.0;
      if (FUSED) sq = load_stamp(N, a.data + o, RESID ? a.model + o : nullptr, R);
      const float spsf = a.psf[st] * 0.42466090014400953f * a.pscale_inv;
      for (int t = threadIdx.x; t < g.ntab; t += blockDim.x) {
        const double2 ks = a.tab.sinc[t < g.h ? g.h - t : t - g.h];
        atab[t] = (float)(exp(-0.5 * (double)spsf * spsf * ks.x * ks.x) * ks.y);
      }
      const float2* dh;
      const float* sqw = nullptr;
      if constexpr (FUSED) {
        if (RESID) {
          sq = wave_sum(sq);
          if (lane_id() == 0) red[wave] = sq;
        }
        __syncthreads();
        if (wave == nw - 1) fill_tables(g, sp, atab, X, Ym, Yf, F, dx, dy);
        stamp_dft<U, MX>(N, sp, tab, R, rows, MX && a.noise_ps ? a.noise_ps + o : nullptr, sqw_s);
        dh = reinterpret_cast<const float2*>(R);
        if (MX) sqw = sqw_s;
        __syncthreads();
      } else {
        // each lane reads its own slots, straight from memory
        dh = a.dh + a.bin_off[st];
        if (MX) sqw = a.sqw + a.bin_off[st];
        __syncthreads();
        fill_tables(g, sp, atab, X, Ym, Yf, F, dx, dy);
      }
      if (wave != 0) continue;
      const LaneCols<P> lc = lane_cols<P>(cols);
      sig = a.sigma[st];
      const float norm = 1.0f / ((float)N * (float)N * sig * sig);
      const KSums S = kspace_sums<PROF, P, RESID, true, 0, 1, 1, MX>(g, sp, lc, dh, X, Ym, Yf, sh, scratch, 0,
                                                                     nullptr, sqw);
      const KResult q = kspace_finish<PROF>(S, sh, F, s, e1, e2, norm);
      r.loglik += q.loglik;
      r.dF += q.dF;
      r.ds += q.ds;
      r.de1 += q.de1;
      r.de2 += q.de2;
      r.ddx += q.ddx;
      r.ddy += q.ddy;
    }
    if (wave != 0) continue;
    uint32_t st = 0;
    if (!(E < 1.0f) || !(s > 0.0f) || !(F > 0.0f)) st |= 1u;
    if (RESID) {
      double chi2 = FUSED ? 0.0 : a.chi2[gal];
      if (FUSED)
        for (int w = 0; w < nw; ++w) chi2 += red[w];
      r.loglik = -0.5 * chi2 / ((double)sig * (double)sig);
    }
    if (!isfinite(r.loglik)) st |= 2u;
    if (threadIdx.x == 0) {
      if (a.loglik) a.loglik[gal] = r.loglik;
      if (a.status) a.status[gal] = st;
    }
    if (a.grad && threadIdx.x < 6) {
      const float v[6] = {r.dF, r.ds, r.de1, r.de2, r.ddx, r.ddy};
      float o = v[0];
#pragma unroll
      for (int j = 1; j < 6; ++j) o = (threadIdx.x == j) ? v[j] : o;
      a.grad[6 * (int64_t)gal + threadIdx.x] = o;
    }
  }
}

template <int PROF, bool RESID, bool MX, int U>
void launch_loglik_u(const LoglikArgs& a, hipStream_t s) {
  const size_t lds = loglik_lds(a.N, a.P, MX, U > 0).total;
  const int nw = U > 0 ? dft_waves(a.N) : 1;
  const dim3 grid(U > 0 ? dft_grid(a.n, nw, lds, loglik_simd_waves(a.P, MX, U)) : a.n), block(kWave * nw);
  auto go = [&](auto kern) {
    if (lds > 64 * 1024)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, block, lds, s, a);
  };
  switch (a.P) {
    case 1: go(loglik_kernel<PROF, RESID, 1, MX, U>); break;
    case 2: go(loglik_kernel<PROF, RESID, 2, MX, U>); break;
    case 3: go(loglik_kernel<PROF, RESID, 3, MX, U>); break;
    case 4: go(loglik_kernel<PROF, RESID, 4, MX, U>); break;
    case 5: go(loglik_kernel<PROF, RESID, 5, MX, U>); break;
    case 6: go(loglik_kernel<PROF, RESID, 6, MX, U>); break;
    default: go(loglik_kernel<PROF, RESID, 8, MX, U>); break;
  }
}

template <int PROF, bool RESID, bool MX>
void launch_loglik_p(const LoglikArgs& a, hipStream_t s) {
  if (!a.data) launch_loglik_u<PROF, RESID, MX, 0>(a, s);
  else if (dft_per_wave(a.N) == 1) launch_loglik_u<PROF, RESID, MX, 1>(a, s);
  else launch_loglik_u<PROF, RESID, MX, 2>(a, s);
}

}  // namespace

// One kernel wherever its waves hold one unit of the transform (up to 63 px):
// 53 px, 1 stamp 19 us against 32 in two kernels, 1,000 27 / 44, 10,000 183 /
// 184 (calls, host included).  Larger stamps leave one or two of its
// workgroups per compute unit, which idle while one wave contracts: 73 px,
// 1,000 stamps 65 / 75 us, 2,000 117 / 116, 4,000 220 / 204; 101 px, 500 73 / 88,
// 1,000 136 / 139, 2,000 253 / 232.
bool loglik_fused(int N, int P, bool mx, int stamps) {
  return !dft_big(N) && loglik_lds(N, P, mx, true).total <= kMaxLds && (dft_per_wave(N) == 1 || stamps <= 1024);
}

hipError_t launch_loglik(LoglikArgs a, int prof, bool resid, bool mx, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (!plan_valid(a.N, a.P)) return hipErrorInvalidValue;
  if (mx && (resid || a.n_exp < 1)) return hipErrorInvalidValue;
  if (loglik_lds(a.N, a.P, mx, a.data != nullptr).total > kMaxLds) return hipErrorInvalidValue;
  a.tab = dft_tables(a.N);
  if (!a.tab.dft) return hipErrorInvalidValue;
  auto run = [&](auto prof_tag) {
    constexpr int PR = decltype(prof_tag)::value;
    if (mx)
      launch_loglik_p<PR, false, true>(a, s);
    else if (resid)
      launch_loglik_p<PR, true, false>(a, s);
    else
      launch_loglik_p<PR, false, false>(a, s);
  };
  if (prof == kProfExp)
    run(std::integral_constant<int, kProfExp>());
  else if (prof == kProfSpergel)
    run(std::integral_constant<int, kProfSpergel>());
  else
    run(std::integral_constant<int, kProfGauss>());
  return hipGetLastError();
}

}  // namespace bsi
