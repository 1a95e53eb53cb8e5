// Chain diagnostics of Section 4.1 over stored samples [gal][C][S][P]: the
// statistics of ess_device.h (multi-chain ESS by Geyer's initial monotone
// sequence, classic and split R-hat) for every galaxy and parameter.
//
// A workgroup holds one galaxy (up to 8 of its parameters), one wave per
// parameter.  The chains pass through LDS one after another as they lie in
// memory, [S][P], the next one's transfer (straight into LDS) under the
// current one's arithmetic.  Of a chain, lane l of the parameter's wave takes
// draws 17 l .. 17 l + 16 (mod 1,088; fewer for short chains) and the 15 after
// them as centred float64
// registers and adds the products at 16 lags at once, 272 multiply-adds for
// 32 LDS reads, into sums that run over the chains; the mean is the only
// thing needed per chain beforehand.  (17 draws: with six parameters the
// lanes' reads are 102 words apart, two lanes to a bank.)  One reduction per
// 16 lags, then the Geyer scan, which for a sampler's draws mostly ends within
// the first 16; each further 16 lags read the chains again.
//
// Bound by vector issue (half of it busy: 5,000 instructions per series, of
// which 1,088 are the products; two workgroups of six waves per compute
// unit).  10,000 galaxies x 4 chains x 1,000 draws x 6 parameters (960 MB):
// 990 us with split R-hat, 820 without; one workgroup per galaxy and
// parameter with its draws read at stride P, 64 lags at least and two LDS
// reads per product took 4,540 us with it.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "bsi_kernels.h"
#include "ess_device.h"

namespace bsi {

namespace {

constexpr int kLags = 16;          // lags per pass over the chains
constexpr int kMaxRun = 17;        // consecutive draws per lane at most
constexpr int kMaxPar = 8;         // parameters (waves) per workgroup
constexpr int kMaxParts = 8;       // waves per parameter
constexpr int kEssChains = 16;     // chains at most
// Series up to which a series' chains are shared by several waves, one parameter
// per workgroup: with fewer waves than the chip holds, the latency of a
// wave's chains one after another counts, not the reads at stride P.
constexpr int64_t kFewSeries = 3072;
constexpr size_t kEssLds = 150 * 1024;   // (ess_buf(S, 1) of the longest chains the entry point takes fits)
constexpr int kWaitVmcnt0 = 0x0F70;   // every vector memory operation done (gfx9 wait counter)

// LDS floats of a chain of S draws at q floats each: the lanes read up to a
// window past the last draw (masked), the transfer writes up to a wave.
__host__ __device__ constexpr int ess_buf(int S, int q) {
  const int tail = (kMaxRun + kLags) * q;
  return (S * q + (tail > kWave ? tail : kWave) + 3) & ~3;
}

// Totals over the wave of 16 per-lane values: value t on lanes 4 t .. 4 t + 3.
__device__ __forceinline__ double wave_total16(double* v) {
  const int lane = lane_id();
#pragma unroll
  for (int n = 8; n >= 1; n >>= 1) {
    const bool up = (lane & (4 * n)) != 0;
#pragma unroll
    for (int j = 0; j < n; ++j) {
      const double send = up ? v[j] : v[j + n], keep = up ? v[j + n] : v[j];
      v[j] = keep + __shfl_xor(send, 4 * n, kWave);
      __builtin_amdgcn_sched_barrier(0);   // one exchange's values live at a time
    }
  }
  double x = v[0];
  x += __shfl_xor(x, 2, kWave);
  x += __shfl_xor(x, 1, kWave);
  return x;
}

// Pooled variance of M <= 32 chains of n draws from the within-chain one W and
// the chains' means.
__device__ __forceinline__ double var_plus(double W, const double* mean, int M, double n) {
  const bool in = lane_id() < M;
  const double x = in ? mean[lane_id()] : 0.0, mm = wave_total(x) / M;
  const double d = in ? x - mm : 0.0;
  const double B = wave_total(d * d);
  return W * (n - 1.0) / n + (M > 1 ? B / (M - 1.0) : 0.0);
}

// q parameters per workgroup, q floats per draw in LDS (q = P: a chain as it
// lies in memory); two buffers, or one.  parts > 1: the chains are shared by
// so many waves per parameter, wave (part j, parameter w) taking chains j,
// j + parts, ... through buffers of its part's own.
template <int q, int kRun>
__global__ void __launch_bounds__(q > 1 ? kWave * q : kWave * kMaxParts, q > 4 ? 4 : 2)
    ess_kernel(int C, int S, int P, int nparts, int buffers, double tau_min, const float* __restrict__ x,
               float* __restrict__ ess, float* __restrict__ rhat, float* __restrict__ rsplit) {
  extern __shared__ float4 ess_lds4[];
  __shared__ double mean_s[q][kEssChains], half_s[q][2 * kEssChains];
  __shared__ double part_s[kMaxParts][kLags + 1];      // parts > 1 (q = 1): each part's sums
  float* lds = reinterpret_cast<float*>(ess_lds4);
  const int groups = (P + q - 1) / q;
  const int gal = blockIdx.x / groups, p0 = (blockIdx.x - gal * groups) * q;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int w = q == 1 ? 0 : wave, part = q == 1 ? wave : 0, parts = q == 1 ? nparts : 1;
  const int size = ess_buf(S, q);
  const float* src = x + (int64_t)gal * C * S * P;
  const int rounds = (C + parts - 1) / parts;
  auto buffer = [&](int r) { return lds + (part * buffers + (buffers == 2 ? r & 1 : 0)) * size; };
  // start the transfer of this part's chain of round r
  auto fetch = [&](int r) {
    const int c = r * parts + part;
    if (c >= C) return;
    float* dst = buffer(r);
    const float* sc = src + (int64_t)c * S * P;
    const int n = S * q;
    for (int i = w * kWave; i < n; i += q * kWave) {
      const int k = min(i + lane, n - 1);
      const int64_t o = q == P ? k : (int64_t)(k / q) * P + min(p0 + k % q, P - 1);
      __builtin_amdgcn_global_load_lds(sc + o, dst + i, 4, 0, 0);
    }
  };
  const int h = S / 2;
  double W = 0.0, vp = 0.0, prev = 1e300, tau_sum = 0.0;   // the same in every lane
  double q2 = 0.0;      // this lane's squared deviations from the half-chain means
  bool done = p0 + w >= P;

  // chain c's mean, and its halves' means and squared deviations (draws [0, h)
  // and [S - h, S); the middle draw of an odd S is in neither)
  auto moments = [&](int c, const float* col) {
    double sa = 0.0, sb = 0.0;
#pragma clang loop unroll(disable)
    for (int s = kRun * lane; s < S; s += kRun * kWave) {
      const int na = h - s, nb = S - h - s, nv = S - s;
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        const float f = col[(s + j) * q];
        sa += (double)(j < na ? f : 0.f);
        sb += (double)((j >= nb) & (j < nv) ? f : 0.f);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    sa = wave_total(sa);
    sb = wave_total(sb);
    const double st = (S & 1) ? sa + sb + (double)col[h * q] : sa + sb;
    if (lane == 0) mean_s[w][c] = st / S;
    if (rsplit) {
      const double ma = sa / h, mb = sb / h;
#pragma clang loop unroll(disable)
      for (int s = kRun * lane; s < S; s += kRun * kWave) {
        const int na = h - s, nb = S - h - s, nv = S - s;
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
          const bool in = (j < na) | ((j >= nb) & (j < nv));
          const double d = in ? (double)col[(s + j) * q] - (j < na ? ma : mb) : 0.0;
          q2 = fma(d, d, q2);
          if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (lane == 0) {
        half_s[w][2 * c] = ma;
        half_s[w][2 * c + 1] = mb;
      }
    }
    wave_lds_sync();
  };

  // lags 16 m .. 16 m + 15 over every chain, and the Geyer scan's next 8 pairs
  // (FIRST: m = 0, with the moments and R-hats)
  auto pass = [&](auto first, int m) {
    constexpr bool FIRST = decltype(first)::value;
    double acc[kLags];
#pragma unroll
    for (int t = 0; t < kLags; ++t) acc[t] = 0.0;
    if (buffers == 2) fetch(0);
#pragma clang loop unroll(disable)
    for (int r = 0; r < rounds; ++r) {
      if (buffers == 1) {
        __syncthreads();     // the last chain has been read
        fetch(r);
      }
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      __syncthreads();       // this round's chains are there, and the other buffers have been read
      if (buffers == 2 && r + 1 < rounds) fetch(r + 1);
      const int c = r * parts + part;
      if (done || c >= C) continue;
      const float* col = buffer(r) + w;
      if (FIRST) moments(c, col);
      const double mean = mean_s[w][c];
      // runs whose every product is past the chain's end are skipped
#pragma clang loop unroll(disable)
      for (int s = kRun * lane; s + kLags * m < S; s += kRun * kWave) {
        const int nv = S - s - kLags * m;
        const float* at = col + s * q;
        const float* to = at + kLags * m * q;
        double y[kRun + kLags - 1];
        // a rolling window: y[j] is dead after draw j
#pragma unroll
        for (int j = 0; j < kRun + kLags - 1; ++j) {
          y[j] = j < nv ? (double)to[j * q] - mean : 0.0;
          const int d = j - (kLags - 1);
          if (d >= 0) {
            const double a = FIRST ? y[d] : (double)at[d * q] - mean;
#pragma unroll
            for (int t = 0; t < kLags; ++t) acc[t] = fma(a, y[d + t], acc[t]);
          }
          if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (done && parts == 1) return;
    double tot = wave_total16(acc);      // lag 16 m + lane / 4
    if (parts > 1) {
      // every part's wave adds the parts' sums in their order and goes on alike
      const double mine = FIRST && rsplit ? wave_total(q2) : 0.0;
      if ((lane & 3) == 0) part_s[part][lane >> 2] = tot;
      if (lane == 1) part_s[part][kLags] = mine;
      __syncthreads();
      tot = 0.0;
      q2 = 0.0;
      for (int j = 0; j < parts; ++j) {
        tot += part_s[j][lane >> 2];
        if (lane == 0) q2 += part_s[j][kLags];
      }
      __syncthreads();
    }
    if (done) return;
    if (FIRST) {
      W = bcast(tot, 0) / ((S - 1.0) * C);
      vp = var_plus(W, mean_s[w], C, S);
      double w2 = 0.0, v2 = 0.0;
      if (rsplit) {
        w2 = wave_total(q2) / ((h - 1.0) * (2 * C));
        v2 = var_plus(w2, half_s[w], 2 * C, h);
      }
      // R-hat on lane 0, split R-hat on lane 1
      float* o = part > 0 ? nullptr : lane == 0 ? rhat : lane == 1 ? rsplit : nullptr;
      if (o) o[(int64_t)gal * P + p0 + w] = (float)sqrt(lane == 0 ? vp / W : v2 / w2);
      done = !(vp > 0.0);
    }
    const double rho = (FIRST && lane < 4) ? 1.0 : 1.0 - (W - tot / ((double)S * C)) / vp;
#pragma unroll
    for (int k = 0; k < kLags / 2; ++k) {
      double Pk = bcast(rho, 8 * k) + bcast(rho, 8 * k + 4);
      if (done || kLags * m + 2 * k + 1 >= S || Pk <= 0.0) {
        done = true;
      } else {
        if (Pk > prev) Pk = prev;
        prev = Pk;
        tau_sum += Pk;
      }
    }
    if (kLags * (m + 1) >= S) done = true;
    if (done && ess && part == 0 && lane == 0) {
      const double n = (double)C * S;
      double tau = (vp > 0.0 && tau_sum > 0.0) ? -1.0 + 2.0 * tau_sum : 1.0;
      tau = fmax(tau, tau_min);
      ess[(int64_t)gal * P + p0 + w] = (vp > 0.0) ? (float)(n / tau) : (float)n;
    }
  };
  pass(std::true_type(), 0);
#pragma clang loop unroll(disable)
  for (int m = 1; __syncthreads_or(!done); ++m) pass(std::false_type(), m);
}

}  // namespace

hipError_t launch_ess(int n_gal, int C, int S, int P, const float* samples, float* ess,
                      float* rhat, float* rsplit, hipStream_t s) {
  if (n_gal <= 0) return hipSuccess;
  if (C > kEssChains) return hipErrorInvalidValue;
  // the parameters (at most 8) whose draws of one chain fit LDS; a second
  // buffer where two workgroups of them still fit a compute unit (1,600 draws
  // of six parameters)
  int q = std::min(P, kMaxPar), parts = 1;
  while (q > 1 && sizeof(float) * (size_t)ess_buf(S, q) > kEssLds) --q;
  // few series: a workgroup each; of one chain only up to about 2 M draws in
  // all, beyond which the strided reads cost more (C = 1, six parameters, a
  // parameter / a galaxy per workgroup: 100 x 200 draws 10.1 / 10.8 us, 100 x 2,000
  // 18.2 / 24.1, 500 x 500 15.1 / 15.7, 200 x 2,000 26.0 / 24.5)
  const int64_t series = (int64_t)n_gal * P;
  if (series <= kFewSeries && (C > 1 || series * S <= 2'000'000)) {
    q = 1;
    parts = std::min(C, kMaxParts);
    while (parts > 1 && parts * sizeof(float) * (size_t)ess_buf(S, 1) > kEssLds) --parts;
  }
  const size_t buf = parts * sizeof(float) * (size_t)ess_buf(S, q);
  const int buffers = buf <= 40 * 1024 ? 2 : 1;
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(buffers * buf));
    hipLaunchKernelGGL(kern, dim3(n_gal * ((P + q - 1) / q)), dim3(kWave * q * parts), buffers * buf, s, C, S, P,
                       parts, buffers, 1.0 / std::log10((double)C * S), samples, ess, rhat, rsplit);
  };
  // the shortest run with which one round of the wave's lanes takes a chain
  // (a wave's time goes with the run, not with the draws); odd, so that the
  // lanes' LDS reads fall on different banks
  auto run = [&](auto qc) {
    constexpr int Q = decltype(qc)::value;
    if (S <= 5 * kWave) go(ess_kernel<Q, 5>);
    else if (S <= 9 * kWave) go(ess_kernel<Q, 9>);
    else go(ess_kernel<Q, kMaxRun>);
  };
  switch (q) {
    case 1: run(std::integral_constant<int, 1>()); break;
    case 2: run(std::integral_constant<int, 2>()); break;
    case 3: run(std::integral_constant<int, 3>()); break;
    case 4: run(std::integral_constant<int, 4>()); break;
    case 5: run(std::integral_constant<int, 5>()); break;
    case 6: run(std::integral_constant<int, 6>()); break;
    case 7: run(std::integral_constant<int, 7>()); break;
    default: run(std::integral_constant<int, 8>()); break;
  }
  return hipGetLastError();
}

}  // namespace bsi
