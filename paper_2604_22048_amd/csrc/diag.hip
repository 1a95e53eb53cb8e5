// Chain diagnostics of Section 4.1 over stored samples [gal][C][S][P]: the
// statistics of ess_device.h (multi-chain ESS by Geyer's initial monotone
// sequence, classic and split R-hat) for every galaxy and parameter.
//
// A workgroup takes one series (the chains of one parameter of one galaxy), all
// its draws in LDS.  The chains are cut into runs of up to 17 draws, dealt to the
// lanes of its waves; a lane takes its run and the 15 draws after it as centred
// float64 registers and adds the products at 16 lags at once, 272 multiply-adds
// for 32 LDS reads.  One reduction per 16 lags, then the Geyer scan, which for a
// sampler's draws mostly ends within the first 16 or 32; slowly mixing chains
// take hundreds, so a pass over further lags costs its products and little else:
// nothing is transferred again, the reduction stays in registers, and where the
// chip has waves to spare several blocks of 16 lags run side by side.
//
// Bound by vector issue.  10,000 galaxies x 4 chains x 1,000 draws x 6 parameters
// (960 MB), a call with split R-hat / without: independent draws 584 / 496 us,
// AR(1) with coefficient 0.5 659 / 579, 0.95 2,840 / 2,710; 30,000 x 4 x 250, 0.95:
// 2,340 / 2,140.  With a galaxy's chains passing through LDS one after another,
// once for every 16 lags, 864 / 700, 1,166 / 1,005, 10,400 / 10,300 and 10,400 /
// 10,200; with 64 lags at once, one to a lane, at two float64 LDS reads a product,
// 4,540 / 3,860, 4,560 / 3,880, 8,960 / 8,280 and 5,490 / 4,010.  A galaxy's
// parameters on one XCD: 855 -> 622 us with split R-hat, the draws at stride P
// being read from memory once.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "bsi_kernels.h"
#include "ess_device.h"

namespace bsi {

namespace {

constexpr int kLags = 16;          // lags per pass over the chains
constexpr int kMaxRun = 17;        // consecutive draws per lane at most
constexpr int kMaxWaves = 8;       // waves per series
constexpr int kSide = 4;           // blocks of 16 lags side by side at most
constexpr int kEssChains = 16;     // chains at most
constexpr int kXcds = 8;

// LDS floats of n draws: the lanes read up to a window past the last one
// (masked), the transfer writes up to a wave.
__host__ __device__ constexpr int ess_buf(int n) { return (n + kWave + 3) & ~3; }
static_assert(kMaxRun + kLags <= kWave, "the window");

// x of the lane DPP names (quad permutations, rotations within 16 lanes).
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffll), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// a (on half the lanes) and b (on the others) added to the same of the lane 32 (or
// 16) further: those halves of the two registers change places.
template <int DIST>
__device__ __forceinline__ double swap_add(double a, double b) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const long long va = __double_as_longlong(a), vb = __double_as_longlong(b);
  u32x2 lo, hi;
  if constexpr (DIST == 32) {
    lo = __builtin_amdgcn_permlane32_swap((unsigned)va, (unsigned)vb, false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)(va >> 32), (unsigned)(vb >> 32), false, false);
  } else {
    lo = __builtin_amdgcn_permlane16_swap((unsigned)va, (unsigned)vb, false, false);
    hi = __builtin_amdgcn_permlane16_swap((unsigned)(va >> 32), (unsigned)(vb >> 32), false, false);
  }
  return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// Totals over the wave of 16 per-lane values: value t on lanes 4 t .. 4 t + 3.
// (Without LDS: through it, an exchange after another, the pass of a short
// chain took longer over this than over its products.)
__device__ __forceinline__ double wave_total16(double* v) {
  const int lane = lane_id();
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = swap_add<32>(v[j], v[j + 8]);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = swap_add<16>(v[j], v[j + 4]);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const bool up = (lane & 8) != 0;
    v[j] = (up ? v[j + 2] : v[j]) + dpp_lane<0x128>(up ? v[j] : v[j + 2]);      // row_ror:8
  }
  const bool up = (lane & 4) != 0;
  double x = (up ? v[1] : v[0]) + __shfl_xor(up ? v[0] : v[1], 4, kWave);
  x += dpp_lane<0x4E>(x);      // quad_perm: lane ^ 2
  x += dpp_lane<0xB1>(x);      // lane ^ 1
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

// Mean of a chain of S draws at col, to mean[c] and, with halves,
// those of its halves (draws [0, h) and [S - h, S); an odd S's middle draw is in
// neither) to half[2 c], half[2 c + 1]; returns q2 plus this lane's squared
// deviations from the latter.  The lane takes runs of kRun draws.
template <int kRun>
__device__ __forceinline__ double moments(const float* col, int S, int c, bool halves, double* mean, double* half,
                                          double q2) {
  const int lane = lane_id(), h = S / 2;
  double sa = 0.0, sb = 0.0;
#pragma clang loop unroll(disable)
  for (int s = kRun * lane; s < S; s += kRun * kWave) {
    const int na = h - s, nb = S - h - s, nv = S - s;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      const float f = col[s + j];
      sa += (double)(j < na ? f : 0.f);
      sb += (double)(((j >= nb) & (j < nv)) ? f : 0.f);
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  sa = wave_total(sa);
  sb = wave_total(sb);
  const double st = (S & 1) ? sa + sb + (double)col[h] : sa + sb;
  if (lane == 0) mean[c] = st / S;
  if (halves) {
    const double ma = sa / h, mb = sb / h;
#pragma clang loop unroll(disable)
    for (int s = kRun * lane; s < S; s += kRun * kWave) {
      const int na = h - s, nb = S - h - s, nv = S - s;
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        const bool in = (j < na) | ((j >= nb) & (j < nv));
        const double d = in ? (double)col[s + j] - (j < na ? ma : mb) : 0.0;
        q2 = fma(d, d, q2);
        if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (lane == 0) {
      half[2 * c] = ma;
      half[2 * c + 1] = mb;
    }
  }
  return q2;
}

// Products of the kRun draws at `at` with those 16 lags on from lag, nv of them
// in the chain (FIRST: lag 0).
template <int kRun, bool FIRST>
__device__ __forceinline__ void lag_products(const float* at, int lag, int nv, double mean, double* acc) {
  const float* to = at + lag;
  double y[kRun + kLags - 1];
  // a rolling window: y[j] is dead after draw j
#pragma unroll
  for (int j = 0; j < kRun + kLags - 1; ++j) {
    y[j] = j < nv ? (double)to[j] - mean : 0.0;
    const int d = j - (kLags - 1);
    if (d >= 0) {
      const double a = FIRST ? y[d] : (double)at[d] - mean;
#pragma unroll
      for (int t = 0; t < kLags; ++t) acc[t] = fma(a, y[d + t], acc[t]);
    }
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// A series' statistics from its lag sums, the same in every lane (of every wave).
struct Series {
  double W, vp, per_n, per_vp, prev, tau_sum;
  bool done;

  // From the sum at lag 0 and the squared deviations from the half-chain means:
  // variances, and R-hat and split R-hat to o_r and o_s.
  __device__ __forceinline__ void start(double tot0, double q2, int C, int S, const double* mean, const double* half,
                                        float* o_r, float* o_s) {
    const int h = S / 2;
    prev = 1e300;
    tau_sum = 0.0;
    W = tot0 / ((S - 1.0) * C);
    vp = var_plus(W, mean, C, S);
    per_n = 1.0 / ((double)S * C);
    per_vp = 1.0 / vp;
    done = !(vp > 0.0);
    if (o_r && lane_id() == 0) *o_r = (float)sqrt(vp / W);
    if (o_s) {
      const double w2 = q2 / ((h - 1.0) * (2 * C)), v2 = var_plus(w2, half, 2 * C, h);
      if (lane_id() == 0) *o_s = (float)sqrt(v2 / w2);
    }
  }

  // The 8 pairs of lags from lag on, the sum at lag + t on lanes 4 t.
  __device__ __forceinline__ void scan(double tot, int lag, int S) {
    const double rho = (lag == 0 && lane_id() < 4) ? 1.0 : 1.0 - (W - tot * per_n) * per_vp;
#pragma unroll
    for (int k = 0; k < kLags / 2; ++k) {
      double Pk = bcast(rho, 8 * k) + bcast(rho, 8 * k + 4);
      if (done || lag + 2 * k + 1 >= S || Pk <= 0.0) {
        done = true;
      } else {
        if (Pk > prev) Pk = prev;
        prev = Pk;
        tau_sum += Pk;
      }
    }
    if (lag + kLags >= S) done = true;
  }

  __device__ __forceinline__ float ess(int C, int S, double tau_min) const {
    const double n = (double)C * S;
    double tau = (vp > 0.0 && tau_sum > 0.0) ? -1.0 + 2.0 * tau_sum : 1.0;
    tau = fmax(tau, tau_min);
    return (vp > 0.0) ? (float)(n / tau) : (float)n;
  }
};

// One series per workgroup, [C][S] in LDS.  Workgroups go to the XCDs in turn: a
// galaxy's parameters, whose draws share memory lines, go to the same one.
template <int kRun>
__global__ void __launch_bounds__(kWave * kMaxWaves, 3)
    ess_kernel(int n_gal, int C, int S, int P, double tau_min, const float* __restrict__ x, float* __restrict__ ess,
               float* __restrict__ rhat, float* __restrict__ rsplit) {
  extern __shared__ float4 ess_lds4[];
  __shared__ double mean_s[kEssChains], half_s[2 * kEssChains], q2_s[kMaxWaves];
  __shared__ double part_s[2][kMaxWaves][kLags];
  float* col = reinterpret_cast<float*>(ess_lds4);
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), T = blockDim.x / kWave;
  const int CS = C * S;
  const unsigned b = blockIdx.x / kXcds;
  const int gal = (int)(b / P) * kXcds + (int)(blockIdx.x % kXcds), par = (int)(b % P);
  if (gal >= n_gal) return;
  const int64_t k = (int64_t)gal * P + par;
  const float* src = x + (int64_t)gal * CS * P + par;
  for (int i = w * kWave; i < CS; i += T * kWave)
    __builtin_amdgcn_global_load_lds(src + (int64_t)min(i + lane, CS - 1) * P, col + i, 4, 0, 0);
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  __syncthreads();
  double q2 = 0.0;
  for (int c = w; c < C; c += T) q2 = moments<kRun>(col + c * S, S, c, rsplit != nullptr, mean_s, half_s, q2);
  if (rsplit) {
    q2 = wave_total(q2);
    if (lane == 0) q2_s[w] = q2;
  }
  __syncthreads();
  // this wave's sums at lags lag .. lag + 15 over the runs whose products reach
  // into their chain, dealt chain by chain to the lanes of `of` waves
  auto sums = [&](auto first, int lag, int part, int of) {
    constexpr bool FIRST = decltype(first)::value;
    const int runs = max((S - lag + kRun - 1) / kRun, 0), items = C * runs;
    const unsigned inv = runs > 1 ? 0xffffffffu / runs + 1 : 0;      // (exact: items runs < 2^32)
    double acc[kLags];
#pragma unroll
    for (int t = 0; t < kLags; ++t) acc[t] = 0.0;
#pragma clang loop unroll(disable)
    for (int i = part * kWave + lane; i < items; i += of * kWave) {
      const int c = runs > 1 ? (int)__umulhi((unsigned)i, inv) : i, s = (i - c * runs) * kRun;
      lag_products<kRun, FIRST>(col + c * S + s, lag, S - lag - s, mean_s[c], acc);
    }
    return wave_total16(acc);
  };
  int round = 0;
  // every wave's sums to LDS, in turn in two places: a barrier per round
  auto share = [&](double tot) {
    if ((lane & 3) == 0) part_s[round & 1][w][lane >> 2] = tot;
    __syncthreads();
  };
  // every wave adds the waves' sums in their order and goes on alike
  auto added = [&](int j0, int step) {
    double tot = 0.0;
    for (int j = j0; j < T; j += step) tot += part_s[round & 1][j][lane >> 2];
    return tot;
  };
  double tot = sums(std::true_type(), 0, w, T);
  if (T > 1) {
    share(tot);
    tot = added(0, 1);
  }
  Series st;
  q2 = 0.0;
  for (int j = 0; rsplit && j < T; ++j) q2 += q2_s[j];
  st.start(bcast(tot, 0), q2, C, S, mean_s, half_s, rhat && w == 0 ? rhat + k : nullptr,
           rsplit && w == 0 ? rsplit + k : nullptr);
  if (!ess) return;
  st.scan(tot, 0, S);
  // further lags: one block of 16 by all waves, then twice as many side by side
  // each time; more at once where the runs do not fill the waves' lanes
  int side = 1;
  while (2 * side <= min(T, kSide) && C * ((S + kRun - 1) / kRun) <= kWave * (T / (2 * side))) side *= 2;
#pragma clang loop unroll(disable)
  for (int lag = kLags; !st.done;) {
    tot = sums(std::false_type(), lag + w % side * kLags, w / side, T / side);
    if (T == 1) {
      st.scan(tot, lag, S);
    } else {
      ++round;
      share(tot);
#pragma clang loop unroll(disable)
      for (int j = 0; j < side && !st.done; ++j) st.scan(added(j, side), lag + j * kLags, S);
    }
    lag += side * kLags;
    if (2 * side <= min(T, kSide)) side *= 2;
  }
  if (w == 0 && lane == 0) ess[k] = st.ess(C, S, tau_min);
}

// Waves per series and draws per run for n series.  A wave's time goes with its
// rounds of runs (20 instructions a draw and 90 more), its chains' moments and
// what it does once, the call's with the rounds of resident workgroups; the
// constants were fitted to 70 shapes, of which the choice is within 2 % of the
// best on average (10,000 galaxies of 4 x 1,000 draws: 1, 2, 4, 8 waves 875, 814,
// 1,005, 2,020 us; 372 series of 8 x 843: 68, 51, 41, 40).
struct EssPlan {
  int T, run;
  size_t lds;
};

EssPlan ess_plan(int64_t n, int C, int S) {
  EssPlan p{1, kMaxRun, sizeof(float) * (size_t)ess_buf(C * S)};
  const int fit = std::max(1, (int)(160 * 1024 / (p.lds + 4096)));      // workgroups per compute unit
  double best = 1e300;
  // (more waves than the blocks side by side have lanes' worth of runs for are idle)
  const int most = std::min(kMaxWaves, kSide * ((C * ((S + 4) / 5) + kWave - 1) / kWave));
  for (int T = 1; T <= most; T *= 2) {
    // (odd runs, so that the lanes' LDS reads fall on different banks)
    for (int run : {kMaxRun, 9, 5}) {
      double turns = (double)n / (256 * std::min(fit, (run == kMaxRun ? 12 : 16) / T));
      if (turns < 2.0) turns = std::ceil(turns);
      const int rounds = (C * ((S + run - 1) / run) + kWave * T - 1) / (kWave * T);
      const double cost = turns * (rounds * (20.5 * run + 90.0) + 400.0 * ((C + T - 1) / T) + 200.0);
      if (cost <= best) {
        best = cost;
        p.T = T;
        p.run = run;
      }
    }
  }
  return p;
}

}  // namespace

hipError_t launch_ess(int n_gal, int C, int S, int P, const float* samples, float* ess,
                      float* rhat, float* rsplit, hipStream_t s) {
  if (n_gal <= 0) return hipSuccess;
  if (C > kEssChains) return hipErrorInvalidValue;
  const EssPlan p = ess_plan((int64_t)n_gal * P, C, S);
  auto kern = p.run == 5 ? ess_kernel<5> : p.run == 9 ? ess_kernel<9> : ess_kernel<kMaxRun>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
  hipLaunchKernelGGL(kern, dim3((n_gal + kXcds - 1) / kXcds * kXcds * P), dim3(kWave * p.T), p.lds, s, n_gal, C, S, P,
                     1.0 / std::log10((double)C * S), samples, ess, rhat, rsplit);
  return hipGetLastError();
}

}  // namespace bsi
