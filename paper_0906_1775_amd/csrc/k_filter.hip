// Inverse-noise filter N^-1: lag construction, overlap-save spectra and the
// overlap-save transform kernel (gfx950).
//
// Weighting section of the MADmap paper: N^-1 is block diagonal with a
// banded Toeplitz block per stationary interval, (N^-1)_{t,t'} = f(|t-t'|)
// for |t - t'| < n_c.  A band of half-width n_c is applied exactly by a
// circulant of length n_f on a window that starts n_c samples before the
// first wanted output; each transform yields m = n_f - 2 n_c exact outputs
// (the chunked scheme of eq. FFTcomplexity).
//
// Lags (the paper leaves the construction of f from p(f) open): f is the
// inverse DFT over L_K frequencies nu_j = j f_samp / L_K of 1/p(nu_j),
// p = sigma^2 (1 + (f_knee/nu)^alpha) (Algorithm section), 1/p(0) taken as its
// limit, times the Bartlett taper (1 - tau/n_c).  Only tau < n_c is needed, so
// the L_K-point inverse DFT is split as j = r + R q (R = L_K / M):
//   F_r(tau) = sum_q s_{r + R q} e^{-2 pi i q tau / M}   (R transforms of M points, period M in tau)
//   f~(tau)  = (1/L_K) sum_r Re [ e^{-2 pi i r tau / L_K} F_r(tau) ],
// and since s_j = s_{L_K - j} the terms of r and R - r are equal: r = 0 .. R/2 suffice.
#include <type_traits>

#include "fft.hpp"
#include "mm_internal.h"

namespace mm {

// ---------------------------------------------------------------- transform shapes
// (threads, log2 points per thread) of the workgroup transform of 2^LOGN points
// and the log2 of the largest radix
template <int LOGN> struct Shape;
template <> struct Shape<6> { static constexpr int NT = 16, LOGE = 2, LOGR = 2; };
template <> struct Shape<7> { static constexpr int NT = 32, LOGE = 2, LOGR = 2; };
template <> struct Shape<8> { static constexpr int NT = 64, LOGE = 2, LOGR = 2; };
template <> struct Shape<9> { static constexpr int NT = 64, LOGE = 3, LOGR = 3; };
template <> struct Shape<10> { static constexpr int NT = 128, LOGE = 3, LOGR = 3; };
template <> struct Shape<11> { static constexpr int NT = 256, LOGE = 3, LOGR = 3; };
template <> struct Shape<12> { static constexpr int NT = 256, LOGE = 4, LOGR = 4; };
template <> struct Shape<13> { static constexpr int NT = 512, LOGE = 4, LOGR = 4; };
template <> struct Shape<14> { static constexpr int NT = 1024, LOGE = 4, LOGR = 4; };
template <> struct Shape<15> { static constexpr int NT = 1024, LOGE = 5, LOGR = 4; };

constexpr int kMinLogN = 6;
constexpr int kMaxLogNF32 = 15;   // n_f = 2^16
constexpr int kMaxLogNF64 = 14;   // n_f = 2^15

int ols_max_logn(bool fp64) { return fp64 ? kMaxLogNF64 : kMaxLogNF32; }

// ---------------------------------------------------------------- tables
// the last twiddle of the overlap-save inverse: exp(-2 pi i n / (4N)), n < N
template <typename T>
__global__ void k_quarter_table(cx<T>* tab, int N) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  double s, c;
  sincospi((double)n / (double)(2 * (int64_t)N), &s, &c);
  tab[n] = {(T)c, (T)(-s)};
}

hipError_t launch_quarter_table(void* tab, int N, bool fp64, hipStream_t s) {
  const int nb = (N + 255) / 256;
  if (fp64)
    hipLaunchKernelGGL(k_quarter_table<double>, dim3(nb), dim3(256), 0, s, (cx<double>*)tab, N);
  else
    hipLaunchKernelGGL(k_quarter_table<float>, dim3(nb), dim3(256), 0, s, (cx<float>*)tab, N);
  return hipGetLastError();
}

// Workgroup shapes of the overlap-save transform; the autotuner may pick any shape that
// exists for a length and precision.  Variant 0 is 16 points per thread: from 2^10
// points on the transform with wavefront-private inner stages (k_ols_wave.hip; float32 up
// to 2^13, float64 up to 2^14), else Shape<LOGN>.  Variant 9 is the wavefront-private
// transform of 2^14 and 2^15 points in float32.  The others are workgroup transforms with
// an LDS exchange after every pass (fft.hpp):
// variant 1 uses half the threads with twice the points each and radix-32 passes;
// variant 2 is that thread count with radix-16 passes, two butterflies per thread;
// variant 3 is variant 2 with the LDS exchanges split into real and imaginary halves
// (68 KB) and at most 128 VGPRs, so that two workgroups share a CU; variant 4 is 256
// threads x 64 points with radix-32 passes, split and two per CU; variant 5 is 1024
// threads x 16 points with radix-8 passes; variant 6 is variant 5 split, two per CU;
// variant 7 is 512 threads x 32 points with radix-8 passes; variant 8 is variant 5 with
// half exchanges (the lower half of the index space, then the upper half, through an LDS
// buffer of N/2 points), two per CU at 64 VGPRs.  BPC: workgroups per CU the register
// budget is sized for.
template <int NT_, int LOGE_, int LOGR_, bool SPLIT_ = false, int BPC_ = 1, bool HALF_ = false>
struct OlsCfg {
  static constexpr int NT = NT_, LOGE = LOGE_, LOGR = LOGR_, BPC = BPC_;
  static constexpr bool SPLIT = SPLIT_, HALF = HALF_;
  // minimum wavefronts per SIMD asked of the register allocator
  static constexpr int WPE = (BPC_ * NT_ / 256) > 1 ? (BPC_ * NT_ / 256) : 1;
};
template <int LOGN, int V> struct OlsShape : OlsCfg<Shape<LOGN>::NT, Shape<LOGN>::LOGE, Shape<LOGN>::LOGR> {};
template <> struct OlsShape<13, 1> : OlsCfg<256, 5, 5> {};
template <> struct OlsShape<14, 1> : OlsCfg<512, 5, 5> {};
template <> struct OlsShape<14, 2> : OlsCfg<512, 5, 4> {};
template <> struct OlsShape<14, 3> : OlsCfg<512, 5, 4, true, 2> {};
template <> struct OlsShape<14, 4> : OlsCfg<256, 6, 5, true, 2> {};
template <> struct OlsShape<14, 5> : OlsCfg<1024, 4, 3> {};
template <> struct OlsShape<14, 6> : OlsCfg<1024, 4, 3, true, 2> {};
template <> struct OlsShape<14, 7> : OlsCfg<512, 5, 3> {};
template <> struct OlsShape<14, 8> : OlsCfg<1024, 4, 3, false, 2, true> {};
template <> struct OlsShape<15, 1> : OlsCfg<512, 6, 5> {};
template <> struct OlsShape<15, 2> : OlsCfg<1024, 5, 3> {};

bool ols_variant_exists(int logn, bool fp64, int v) {
  if (v == 0) return logn >= kMinLogN && logn <= ols_max_logn(fp64);
  if (v == 9) return !fp64 && (logn == 14 || logn == 15);
  if (v == 5 || v == 7 || (v == 2 && logn == 14)) return logn == 14;
  if (fp64) return false;
  return (v == 1 && (logn == 13 || logn == 14 || logn == 15)) || ((v >= 2 && v <= 6) && logn == 14) ||
         (v == 8 && logn == 14) ||
         (v == 2 && logn == 15);
}

bool ols_variant_wave(int logn, bool fp64, int v) {
  return v == 9 || (v == 0 && logn >= 10 && logn <= (fp64 ? 14 : 13));
}

template <typename T, int LOGN, int V = 0>
using ShapeFFT = BlockFFT<T, LOGN, OlsShape<LOGN, V>::NT, OlsShape<LOGN, V>::LOGE, OlsShape<LOGN, V>::LOGR,
                          OlsShape<LOGN, V>::SPLIT, OlsShape<LOGN, V>::HALF>;

// per-pass twiddle rows: entry (j, r) of pass p = exp(-2 pi i (j + shift) r / (Ns R)), shift
// in the forward sequence only
template <typename T, int LOGN, int V>
__global__ void k_pass_tw(cx<T>* tab, double shift) {
  using F = ShapeFFT<T, LOGN, V>;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= F::tw_total()) return;
  for (int sq = 0; sq < 2; ++sq) {
    const bool fwd = sq == 0;
    for (int p = 0; p < F::NP; ++p) {
      const int o = F::tw_offset(fwd, p), c = F::tw_count(fwd, p);
      if (e >= o && e < o + c) {
        const int lr = F::log_radix(fwd, p), ls = F::log_span(fwd, p);
        const int j = (e - o) >> lr, r = (e - o) & ((1 << lr) - 1);
        const double frac = ((double)j + (fwd ? shift : 0.0)) * (double)r / (double)(1 << (lr + ls));
        double sn, cs;
        sincospi(2.0 * frac, &sn, &cs);
        tab[e] = {(T)cs, (T)(-sn)};
        return;
      }
    }
  }
}

// Calls f(F, V) with the workgroup transform type of 2^logn points in variant v (which
// must exist and not be a wavefront-private one), else returns `none`
template <typename T, typename R, typename Fn>
static R with_shape(int logn, int v, R none, Fn f) {
#define MM_SHAPE(L, V) return f(std::integral_constant<int, L>{}, std::integral_constant<int, V>{})
  if (logn == 14) {
    if (v == 2) MM_SHAPE(14, 2);
    if (v == 5) MM_SHAPE(14, 5);
    if (v == 7) MM_SHAPE(14, 7);
  }
  if constexpr (sizeof(T) == 4) {
    if (logn == 13 && v == 1) MM_SHAPE(13, 1);
    if (logn == 14) {
      if (v == 0) MM_SHAPE(14, 0);
      if (v == 1) MM_SHAPE(14, 1);
      if (v == 3) MM_SHAPE(14, 3);
      if (v == 4) MM_SHAPE(14, 4);
      if (v == 6) MM_SHAPE(14, 6);
      if (v == 8) MM_SHAPE(14, 8);
    }
    if (logn == 15) {
      if (v == 0) MM_SHAPE(15, 0);
      if (v == 1) MM_SHAPE(15, 1);
      if (v == 2) MM_SHAPE(15, 2);
    }
  }
  if (v == 0) {
    if (logn == 6) MM_SHAPE(6, 0);
    if (logn == 7) MM_SHAPE(7, 0);
    if (logn == 8) MM_SHAPE(8, 0);
    if (logn == 9) MM_SHAPE(9, 0);
  }
#undef MM_SHAPE
  return none;
}

int pass_twiddle_count(int logn, bool fp64, int variant) {
  if (!ols_variant_exists(logn, fp64, variant)) return -1;
  if (ols_variant_wave(logn, fp64, variant)) return ols_wave_table_count(logn);
  auto go = [&](auto tc) {
    using T = decltype(tc);
    return with_shape<T>(logn, variant, -1, [](auto L, auto V) -> int {
      return ShapeFFT<T, decltype(L)::value, decltype(V)::value>::tw_total();
    });
  };
  return fp64 ? go(double{}) : go(float{});
}

template <typename T, int LOGN, int V = 0>
static hipError_t pass_tw_launch(void* tab, double shift, hipStream_t s) {
  const int n = ShapeFFT<T, LOGN, V>::tw_total();
  hipLaunchKernelGGL((k_pass_tw<T, LOGN, V>), dim3((n + 255) / 256), dim3(256), 0, s, (cx<T>*)tab, shift);
  return hipGetLastError();
}

hipError_t launch_pass_twiddles(void* tab, int logn, bool fp64, hipStream_t s, int variant) {
  if (!ols_variant_exists(logn, fp64, variant)) return hipErrorInvalidValue;
  if (ols_variant_wave(logn, fp64, variant)) return launch_wave_tables(logn, fp64, tab, s);
  auto go = [&](auto tc) {
    using T = decltype(tc);
    return with_shape<T>(logn, variant, hipErrorInvalidValue, [&](auto L, auto V) -> hipError_t {
      return pass_tw_launch<T, decltype(L)::value, decltype(V)::value>(tab, 0.25, s);
    });
  };
  return fp64 ? go(double{}) : go(float{});
}

// plain float64 transforms of the lags and the symbols: tables of Shape<logn>
template <typename Fn>
static auto with_plain(int logn, Fn f) {
#define MM_PLAIN(L) case L: return f(std::integral_constant<int, L>{});
  switch (logn) {
    MM_PLAIN(6) MM_PLAIN(7) MM_PLAIN(8) MM_PLAIN(9) MM_PLAIN(10) MM_PLAIN(11) MM_PLAIN(12) MM_PLAIN(13)
    default: return f(std::integral_constant<int, 14>{});
  }
#undef MM_PLAIN
}
static int plain_twiddle_count(int logn) {
  return with_plain(logn, [](auto L) -> int { return ShapeFFT<double, decltype(L)::value>::tw_total(); });
}
static hipError_t launch_plain_twiddles(void* tab, int logn, hipStream_t s) {
  return with_plain(logn, [&](auto L) -> hipError_t { return pass_tw_launch<double, decltype(L)::value>(tab, 0.0, s); });
}

// log2 of the fraction of j: tab[j] = log2(j / 2^e), 2^e <= j < 2^(e + 1), j = 1 .. n - 1
__device__ __forceinline__ double log2_fraction(uint32_t j, int e) {
  return log2((double)j * __builtin_bit_cast(double, (uint64_t)(1023 - e) << 52));
}
__global__ void k_log2_table(double* __restrict__ tab, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j == 0 || j >= n) return;
  tab[j] = log2_fraction((uint32_t)j, 31 - __clz((uint32_t)j));
}

// Noise parameters of one filter, with q = f_knee L / f_samp split as 2^e2 times a fraction
struct PsdParams {
  double sigma, fknee, alpha, frac2;
  int e2;
};
__device__ __forceinline__ PsdParams psd_params(const double* __restrict__ p, double f_samp, int64_t L) {
  PsdParams P{p[0], p[1], p[2], 0.0, 0};
  if (P.fknee != 0.0) P.frac2 = log2(frexp(P.fknee * ((double)L / f_samp), &P.e2));
  return P;
}

// 1/p(nu_j) on the L-point grid, Hermitian-extended: s_j = s_{L-j}; mode 1-3
// give its derivative with respect to sigma, f_knee, alpha.  With
// x = (f_knee/nu)^alpha:  ds/dsigma = -2 s/sigma,  ds/df_knee = -s^2 sigma^2 alpha x/f_knee,
// ds/dalpha = -s^2 sigma^2 x ln(f_knee/nu); the nu = 0 value (0 or 1/sigma^2)
// does not depend on f_knee or alpha.
// x = 2^(alpha log2(f_knee / nu_j)) with log2(f_knee L / f_samp) - log2(j) held as an integer
// and a fraction, and the product's rounding carried to first order, so that x is as
// accurate as pow(f_knee / nu, alpha) (whose argument is rounded, an error times alpha) at
// a fifth of its operations.
__device__ __forceinline__ double inv_psd(uint32_t j, uint32_t L, const PsdParams& P, const double* __restrict__ tab,
                                          int mode) {
  const double sigma = P.sigma, fknee = P.fknee, alpha = P.alpha;
  if (j > L / 2) j = L - j;
  if (j == 0) {
    const double s0 = fknee > 0.0 ? 0.0 : 1.0 / (sigma * sigma);
    return mode == 0 ? s0 : (mode == 1 ? -2.0 * s0 / sigma : 0.0);
  }
  double x = 0.0, ln = 0.0;
  if (fknee != 0.0) {
    const int e = 31 - __clz(j);
    const double di = (double)(P.e2 - e), df = P.frac2 - (tab ? tab[j] : log2_fraction(j, e));
    const double hi = alpha * di, v = fma(alpha, df, fma(alpha, di, -hi));
    const double w = hi + v, rest = v - (w - hi);
    x = exp2(w);
    if (isfinite(x)) x = fma(x * 0.69314718055994530942, rest, x);
    ln = (di + df) * 0.69314718055994530942;
  }
  const double s = 1.0 / (sigma * sigma * (1.0 + x));
  switch (mode) {
    case 0: return s;
    case 1: return -2.0 * s / sigma;
    case 2: return fknee > 0.0 ? -s * s * sigma * sigma * alpha * x / fknee : 0.0;
    default: return fknee > 0.0 ? -s * s * sigma * sigma * x * ln : 0.0;
  }
}

// Partial sums over r of the lags: grid (G groups, filters in batch); group g takes
// r = g, g + G, .. <= R/2, keeps its sums over tau < NB M in registers and writes them to
// part[filter][g][tau].  Every F_r stays on chip (written out and read back they were 16 bytes
// per frequency and filter, and the sum over r ran serially in n_c threads).
template <int LOGM, int NB>
__global__ __launch_bounds__(Shape<LOGM>::NT) void k_lag_sums(const double* __restrict__ params, int n_filters, int f0,
                                                              double f_samp, int64_t L, int n_c,
                                                              const cx<double>* __restrict__ ptw,
                                                              const double* __restrict__ tab,
                                                              double* __restrict__ part, int mode0) {
  using F = ShapeFFT<double, LOGM>;
  __shared__ __align__(16) char lds[F::LDS_BYTES];
  constexpr int M = F::N, E = F::E;
  const int t = threadIdx.x;
  const uint32_t R = (uint32_t)(L >> LOGM), mask = (uint32_t)L - 1;   // (L <= 2^30)
  const double unit = 2.0 / (double)L;   // exact: L is a power of two
  const int set = f0 + (int)blockIdx.y, mode = mode0 + set / n_filters;   // sets: filters of mode0, of the next, ..
  const PsdParams P = psd_params(params + 3 * (int64_t)(set % n_filters), f_samp, L);
  constexpr int L0 = F::first_log_fwd(), R0 = 1 << L0;
  constexpr int LL = F::last_log_fwd(), RL = 1 << LL;
  double acc[NB][E];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < E; ++i) acc[b][i] = 0.0;
  for (uint32_t r = blockIdx.x; r <= R / 2; r += gridDim.x) {
    cx<double> v[E];
#pragma unroll
    for (int i = 0; i < E / R0; ++i)
#pragma unroll
      for (int rr = 0; rr < R0; ++rr)
        v[i * R0 + rr] = {inv_psd(r + R * (uint32_t)F::template in_index<L0>(t, i, rr), (uint32_t)L, P, tab, mode), 0.0};
    F::forward(v, lds, ptw, t);
    const double twice = r == 0 || 2 * r == R ? 1.0 : 2.0;
    // e^{-2 pi i r tau / L} F_r(tau): exact at tau < M, then by e^{-2 pi i r / R} per block of M
    cx<double> wr = {1.0, 0.0};
    if (NB > 1) sincospi(unit * (double)(r << LOGM), &wr.im, &wr.re), wr.im = -wr.im;
#pragma unroll
    for (int i = 0; i < E / RL; ++i)
#pragma unroll
      for (int rr = 0; rr < RL; ++rr) {
        const int e = i * RL + rr, tau = t + i * F::NT + rr * (M >> LL);
        double sn, cs;
        sincospi(unit * (double)((r * (uint32_t)tau) & mask), &sn, &cs);
        cx<double> z = cmul(v[e], cx<double>{twice * cs, -twice * sn});
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          acc[b][e] += z.re;
          if (b + 1 < NB) z = cmul(z, wr);
        }
      }
  }
  double* __restrict__ out = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * n_c;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < E / RL; ++i)
#pragma unroll
      for (int rr = 0; rr < RL; ++rr) {
        const int tau = b * M + t + i * F::NT + rr * (M >> LL);
        if (tau < n_c) out[tau] = acc[b][i * RL + rr];
      }
}

// lags[f][tau] = taper * (1/L) sum_g part[f][g][tau]
__global__ void k_lag_reduce(const double* __restrict__ part, int f0, int64_t L, int groups, int n_c,
                             double* __restrict__ lags) {
  const int tau = blockIdx.x * blockDim.x + threadIdx.x;
  if (tau >= n_c) return;
  const double* __restrict__ p = part + (int64_t)blockIdx.y * groups * n_c + tau;
  double acc = 0.0;
#pragma unroll 8
  for (int g = 0; g < groups; ++g) acc += p[(int64_t)g * n_c];
  lags[(int64_t)(f0 + blockIdx.y) * n_c + tau] = acc / (double)L * (1.0 - (double)tau / (double)n_c);
}

static int ceil_log2(int64_t x) {
  int l = 0;
  while ((int64_t(1) << l) < x) ++l;
  return l;
}

static size_t lag_tw_bytes(int logn) {
  return ((size_t)plain_twiddle_count(logn) * sizeof(cx<double>) + 255) & ~(size_t)255;
}
static int lag_min_logm(int n_c) { return ceil_log2(n_c) < kMinLogN ? kMinLogN : ceil_log2(n_c); }

size_t lags_scratch_bytes(int n_c, int64_t lag_len, int filters_per_batch) {
  const int logn = lag_min_logm(n_c);
  const int64_t R = lag_len >> logn;
  return lag_tw_bytes(logn) + (size_t)filters_per_batch * R * n_c * sizeof(cx<double>);
}

// Split of the lag construction, a function of n_c and L alone (the lags then do not depend on
// the scratch a caller gives): M = 2^11 points (four 37 KB workgroups per CU, and at most
// eight blocks of M lags) where L allows, and up to kLagGroups groups of r, so that one
// filter already occupies many CUs, within the scratch of one filter.  L = 2^20, one filter:
// 74 -> 49 us at n_c = 8192, 3,910 -> 46 us at 64 (M was the power of two above n_c, the sum
// over r a serial loop); 64 filters at 8192: 4,690 -> 670 us.  M = 2^13 at n_c = 8192 (one
// workgroup per CU): 126 and 1,139 us.
constexpr int kLagLogM = 11, kLagGroups = 65;
struct LagSplit {
  int logm, groups;
};
static LagSplit lag_split(int n_c, int64_t lag_len) {
  const size_t have = lags_scratch_bytes(n_c, lag_len, 1);
  for (int logm = kLagLogM; logm >= kMinLogN; --logm) {
    const int64_t R = lag_len >> logm;
    if (R < 2 || lag_tw_bytes(logm) >= have) continue;
    const int64_t fit = (int64_t)((have - lag_tw_bytes(logm)) / ((size_t)n_c * sizeof(double)));
    const int64_t want = R / 2 + 1 < kLagGroups ? R / 2 + 1 : kLagGroups;
    // (shorter transforms only where the longer one's tables crowd out its groups)
    if (fit >= want || (fit >= 1 && logm <= lag_min_logm(n_c))) return {logm, (int)(fit < want ? fit : want)};
  }
  return {0, 0};
}

hipError_t launch_lags(const double* params, int n_filters, double f_samp, int n_c,
                       int64_t lag_len, double* lags, void* scratch, size_t scratch_bytes,
                       hipStream_t s, int mode, int n_modes) {
  if (lag_min_logm(n_c) > kMaxLogNF64) return hipErrorInvalidValue;
  const int64_t R0 = lag_len >> lag_min_logm(n_c);
  if (R0 < 2 || (R0 << lag_min_logm(n_c)) != lag_len) return hipErrorInvalidValue;
  if (scratch_bytes < lags_scratch_bytes(n_c, lag_len, 1)) return hipErrorInvalidValue;
  const LagSplit sp = lag_split(n_c, lag_len);
  if (sp.groups < 1 || n_c > (8 << sp.logm)) return hipErrorInvalidValue;
  // scratch: twiddles, the log2 table (where it leaves room for the partial sums of eight
  // filters, or of all; else the kernel evaluates the same logarithms), partial sums
  cx<double>* ptw = (cx<double>*)scratch;
  size_t off = lag_tw_bytes(sp.logm);
  const size_t per_filter = (size_t)sp.groups * n_c * sizeof(double);
  const size_t tab_bytes = ((size_t)(lag_len / 2 + 1) * sizeof(double) + 255) & ~(size_t)255;
  double* tab = nullptr;
  hipError_t e = launch_plain_twiddles(ptw, sp.logm, s);
  if (e != hipSuccess) return e;
  if (off + tab_bytes + (size_t)(n_filters < 8 ? n_filters : 8) * per_filter <= scratch_bytes) {
    tab = (double*)((char*)scratch + off);
    off += tab_bytes;
    const int64_t n = lag_len / 2 + 1;
    hipLaunchKernelGGL(k_log2_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, tab, n);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  double* part = (double*)((char*)scratch + off);
  const size_t fit = (scratch_bytes - off) / per_filter;
  const int batch = (int)(fit < 65535 ? fit : 65535);   // sets per launch (grid y)
  const int n_sets = n_filters * n_modes;
  for (int f0 = 0; f0 < n_sets; f0 += batch) {
    const int nb = (n_sets - f0) < batch ? (n_sets - f0) : batch;
    e = with_plain(sp.logm, [&](auto LC) -> hipError_t {
      constexpr int LOGM = decltype(LC)::value < kLagLogM ? decltype(LC)::value : kLagLogM;
      const dim3 g((unsigned)sp.groups, (unsigned)nb), b(Shape<LOGM>::NT);
#define MM_LAGS(NB) \
  hipLaunchKernelGGL((k_lag_sums<LOGM, NB>), g, b, 0, s, params, n_filters, f0, f_samp, lag_len, n_c, ptw, tab, part, mode)
      if (n_c <= (1 << LOGM)) MM_LAGS(1);
      else if (n_c <= (2 << LOGM)) MM_LAGS(2);
      else if (n_c <= (4 << LOGM)) MM_LAGS(4);
      else MM_LAGS(8);
#undef MM_LAGS
      return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lag_reduce, dim3((unsigned)((n_c + 255) / 256), (unsigned)nb), dim3(256), 0, s, part, f0,
                       lag_len, sp.groups, n_c, lags);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------- spectra
// Symbol of one filter's band at the N frequencies of the shifted transform:
//   F_k = f(0) + 2 sum_{tau=1}^{n_c-1} f(tau) cos(2 pi (k + 1/4) tau / N),  k = 0 .. N - 1.
// The frequencies k = b + B k' (b < B = N / N') are those of an N'-point transform shifted
// by phi = (b + 1/4) / B, so a workgroup per (b, filter) folds the two-sided band
// f(|tau|) exp(-2 pi i tau phi / N') onto N' points, transforms them in float64 and keeps
// the real parts: N' = min(N, 2^12), so that a few filters already occupy many CUs and no
// length is beyond an on-chip transform.  The table keeps F / N in the filter's working
// precision, k in row order: entry (k mod NO) N / NO + k / NO, NO = 2^rowlog rows (the order
// the wavefront-private and the long transforms read it in; NO = 1: natural order).
constexpr int kSymbolLogN = 12;

template <typename T, int LOGM>
__global__ __launch_bounds__(Shape<LOGM>::NT) void k_symbol(
    const double* __restrict__ lags, int n_c, int logn, int rowlog, T* __restrict__ spec,
    const cx<double>* __restrict__ ptw) {
  using F = ShapeFFT<double, LOGM>;
  __shared__ __align__(16) char lds[F::LDS_BYTES];
  constexpr int M = F::N, E = F::E;
  const int t = threadIdx.x;
  const int b = blockIdx.x, B = gridDim.x;
  const uint32_t N = 1u << logn, mask = 4 * N - 1;
  const double unit = 0.5 / (double)N;   // exact: N is a power of two
  const double* __restrict__ f = lags + (int64_t)blockIdx.y * n_c;
  cx<double> v[E];
  constexpr int L0 = F::first_log_fwd(), R0 = 1 << L0;
#pragma unroll
  for (int i = 0; i < E / R0; ++i)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int n = F::template in_index<L0>(t, i, r);
      cx<double> u = {0.0, 0.0};
      // tau = n - M q, |tau| < n_c; tau phi / M = tau (4 b + 1) / (4 N) turns
      for (int q = n < n_c ? -((n_c - 1 - n) / M) : (n - n_c) / M + 1; n - M * q > -n_c; ++q) {
        const int tau = n - M * q;
        double sn, cs;
        sincospi(unit * (double)(((uint32_t)tau * (uint32_t)(4 * b + 1)) & mask), &sn, &cs);
        const double x = f[tau < 0 ? -tau : tau];
        u.re += x * cs;
        u.im -= x * sn;
      }
      v[i * R0 + r] = u;
    }
  F::forward(v, lds, ptw, t);
  const double scale = 1.0 / (double)N;
  T* __restrict__ out = spec + (int64_t)blockIdx.y * (N + 1);
  constexpr int LL = F::last_log_fwd(), RL = 1 << LL;
#pragma unroll
  for (int i = 0; i < E / RL; ++i)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const uint32_t k = (uint32_t)(b + B * (t + i * F::NT + r * (M >> LL)));
      out[((k & ((1 << rowlog) - 1)) << (logn - rowlog)) + (k >> rowlog)] = (T)(v[i * RL + r].re * scale);
    }
}

// A float64 sum with its roundings (Knuth's exact addition)
struct Sum2 {
  double hi, lo;
  __device__ __forceinline__ void add(double x) {
    const double s = hi + x, z = s - hi;
    lo += (hi - (s - z)) + (x - z);
    hi = s;
  }
};

// f(0) + 2 sum_{tau = 1}^{n_c - 1} f(tau) behind each filter's N symbol values, one block per filter.
// It is small beside f(0) (a 1/f filter passes no constant), hence the compensated sums.
template <typename T>
__global__ __launch_bounds__(1024) void k_lag_total(const double* __restrict__ lags, int n_c, int64_t N,
                                                    T* __restrict__ spec) {
  __shared__ double sh[2][1024];
  const int tid = threadIdx.x;
  const double* __restrict__ f = lags + (int64_t)blockIdx.x * n_c;
  Sum2 s{0.0, 0.0};
  for (int64_t tau = tid; tau < n_c; tau += 1024) s.add(tau ? f[tau] : 0.5 * f[0]);
  for (int o = 512; o >= 1; o >>= 1) {
    sh[0][tid] = s.hi;
    sh[1][tid] = s.lo;
    __syncthreads();
    if (tid < o) {
      s.add(sh[0][tid + o]);
      s.lo += sh[1][tid + o];
    }
    __syncthreads();
  }
  if (tid == 0) spec[(int64_t)blockIdx.x * (N + 1) + N] = (T)(2.0 * (s.hi + s.lo));
}

static int symbol_logm(int logn) { return logn < kSymbolLogN ? logn : kSymbolLogN; }

size_t spectra_scratch_bytes(int logn) { return (size_t)plain_twiddle_count(symbol_logm(logn)) * sizeof(cx<double>) + 256; }

hipError_t launch_spectra(const double* lags, int n_filters, int n_c, int logn, int rowlog, bool fp64, void* spec,
                          void* scratch, hipStream_t s) {
  if (n_filters == 0) return hipSuccess;
  if (logn < kMinLogN || rowlog < 0 || rowlog > logn) return hipErrorInvalidValue;
  const int logm = symbol_logm(logn);
  hipError_t e = launch_plain_twiddles(scratch, logm, s);
  if (e != hipSuccess) return e;
  return with_plain(logm, [&](auto L) -> hipError_t {
    constexpr int LOGM = decltype(L)::value <= kSymbolLogN ? decltype(L)::value : kSymbolLogN;
    // (filters along grid y, at most 65535 of them per launch)
    for (int f0 = 0; f0 < n_filters; f0 += 65535) {
      const dim3 g(1u << (logn - LOGM), (unsigned)(n_filters - f0 < 65535 ? n_filters - f0 : 65535));
      const double* lg = lags + (int64_t)f0 * n_c;
      auto go = [&](auto tc) {
        using T = decltype(tc);
        const int64_t N = int64_t(1) << logn;
        T* out = (T*)spec + f0 * (N + 1);
        hipLaunchKernelGGL((k_symbol<T, LOGM>), g, dim3(Shape<LOGM>::NT), 0, s, lg, n_c, logn, rowlog, out,
                           (const cx<double>*)scratch);
        hipLaunchKernelGGL(k_lag_total<T>, dim3(g.y), dim3(1024), 0, s, lg, n_c, N, out);
      };
      if (fp64) go(double{});
      else go(float{});
      const hipError_t el = hipGetLastError();
      if (el != hipSuccess) return el;
    }
    return hipSuccess;
  });
}

// ---------------------------------------------------------------- overlap-save transform
// One workgroup per (chunk, RHS).  The n_f = 2N real window x is z_n = x_n - i x_(n+N)
// (negacyclic embedding, see k_ols_wave.hip): its shifted transform Z meets the real
// symbol F pointwise, and exp(-2 pi i n / (4N)) times the plain transform of
// conj(F Z) is y_n + i y_(n+N), all of it without the window's mean (window_mean).  The table spec
// holds F / N, and behind it the response to a constant.

template <typename T, typename Tin, int LOGN, int V>
__global__ __attribute__((amdgpu_flat_work_group_size(1, OlsShape<LOGN, V>::NT),
                          amdgpu_waves_per_eu(OlsShape<LOGN, V>::WPE))) void k_ols(
    const Tin* __restrict__ yin, T* __restrict__ yout, const OlsChunk* __restrict__ chunks,
    const T* __restrict__ spec, const cx<T>* __restrict__ ptw, const cx<T>* __restrict__ qtw,
    int64_t n_t, int n_c, int m, const CgState* __restrict__ st) {
  using F = ShapeFFT<T, LOGN, V>;
  // Workgroups are dealt to the 8 XCDs round-robin in linear (x-fastest) order, so
  // XCD x takes workgroups x, x + 8, ...; give it a contiguous run of (RHS, chunk)
  // pairs instead, so that neighbouring chunks, whose windows overlap by 2 n_c
  // samples, read the shared samples through the same L2.
  const int64_t n_wg = (int64_t)gridDim.x * gridDim.y;
  const int64_t wl = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t xq = n_wg >> 3, xr = n_wg & 7, xw = wl & 7;
  const int64_t job = xw * xq + (xw < xr ? xw : xr) + (wl >> 3);
  const int rhs = __builtin_amdgcn_readfirstlane((int)(job / gridDim.x));   // uniform: scalar row offsets
  if (st && !st[rhs].active) return;   // this RHS has stopped iterating
  __shared__ __align__(16) char lds[F::LDS_BYTES];
  constexpr int N = F::N, E = F::E, NT = F::NT;
  const int t = threadIdx.x;
  const OlsChunk ch = chunks[job - (int64_t)rhs * gridDim.x];
  const int64_t roff = (int64_t)rhs * n_t;
  const int64_t s0 = ch.out_start - n_c;
  const int64_t lo = ch.iv_lo, hi = ch.iv_hi;

  cx<T> v[E];
  constexpr int L0 = F::first_log_fwd(), R0 = 1 << L0;
  // window samples [a, b) are data; a buffer over them gives zeros elsewhere (see
  // k_ols_wave: the constants beside a thread's offset must not move into the instruction)
  const int a = (int)(lo > s0 ? lo - s0 : 0);   // (lo <= out_start: a <= n_c)
  const int b = (int)(hi - s0 < 2 * N ? hi - s0 : 2 * N);
  const Rsrc src = buffer_of(yin + roff + s0 + a, (b - a) * (int)sizeof(Tin));
  T c = (T)0;
  if constexpr (NT > 64)
    c = window_mean<T, 2 * N>(t, [&](int n) {
      Tin x;
      buffer_get(src, opaque((uint32_t)(n - a) * (uint32_t)sizeof(Tin)), x);
      return (T)x;
    });
#pragma unroll
  for (int i = 0; i < E / R0; ++i)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const uint32_t off = opaque((uint32_t)(F::template in_index<L0>(t, i, r) - a) * (uint32_t)sizeof(Tin));
      Tin x, y;
      buffer_get(src, off, x);
      buffer_get(src, opaque(off + N * (uint32_t)sizeof(Tin)), y);
      v[i * R0 + r] = {(T)x - c, c - (T)y};
    }
  if constexpr (NT <= 64) {   // one wavefront: from all samples
    T sum = (T)0, sq = (T)0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      sum += v[e].re - v[e].im;
      sq += v[e].re * v[e].re + v[e].im * v[e].im;
    }
    c = offset_of<NT>(sum, sq, 2 * N);
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = {v[e].re - c, v[e].im + c};
  }

  F::template forward<true>(v, lds, ptw, t);
  const T* __restrict__ S = spec + (int64_t)ch.filter * (N + 1);
  const T back = c * S[N];   // what the filter makes of the mean
  constexpr int LL = F::last_log_fwd(), RL = 1 << LL;
#pragma unroll
  for (int i = 0; i < E / RL; ++i)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const T f = S[(uint32_t)(t + i * NT + r * (N >> LL))];
      cx<T>& z = v[i * RL + r];
      z = {z.re * f, -(z.im * f)};
    }
  F::forward_rev(v, lds, ptw, t);

  constexpr int LZ = F::last_log_rev(), RZ = 1 << LZ;
  // window positions [n_c, n_c + m) are the chunk's outputs, from out_start on
  const int len = (int)(hi - ch.out_start < m ? hi - ch.out_start : m);   // outputs of this chunk
  const Rsrc dst = buffer_of(yout + roff + ch.out_start, len * (int)sizeof(T));
#pragma unroll
  for (int i = 0; i < E / RZ; ++i)
#pragma unroll
    for (int r = 0; r < RZ; ++r) {
      const int n = t + i * NT + r * (N >> LZ);
      const cx<T> z = cmul(v[i * RZ + r], qtw[n]);
      const uint32_t off = opaque((uint32_t)(n - n_c) * (uint32_t)sizeof(T));   // wraps below n_c
      buffer_put(dst, off, z.re + back);
      buffer_put(dst, opaque(off + N * (uint32_t)sizeof(T)), z.im + back);
    }
}

template <typename T, typename Tin>
static hipError_t ols_dispatch(int logn, int variant, const void* y_in, void* y_out, const OlsChunk* chunks,
                               int n_chunks, const void* spec, const void* ptw, const void* qtw,
                               int64_t n_t, int n_c, int m, int n_rhs, hipStream_t s, const CgState* st) {
  return with_shape<T>(logn, variant, hipErrorInvalidValue, [&](auto L, auto V) -> hipError_t {
    constexpr int LOGN = decltype(L)::value, VV = decltype(V)::value;
    hipLaunchKernelGGL((k_ols<T, Tin, LOGN, VV>), dim3((unsigned)n_chunks, (unsigned)n_rhs),
                       dim3(OlsShape<LOGN, VV>::NT), 0, s, (const Tin*)y_in, (T*)y_out, chunks,
                       (const T*)spec, (const cx<T>*)ptw, (const cx<T>*)qtw, n_t, n_c, m, st);
    return hipGetLastError();
  });
}

hipError_t launch_ols(bool fp64, bool in_f64, int logn, const void* y_in, void* y_out,
                      const OlsChunk* chunks, int n_chunks, const void* spec, const void* ptw,
                      const void* qtw, int64_t n_t, int n_c, int m, int n_rhs, hipStream_t s, int variant,
                      const CgState* st) {
  if (!ols_variant_exists(logn, fp64, variant)) return hipErrorInvalidValue;
  if (n_chunks == 0 || n_rhs == 0) return hipSuccess;
  if (ols_variant_wave(logn, fp64, variant))
    return launch_ols_wave(logn, fp64, in_f64, y_in, y_out, chunks, n_chunks, spec, ptw, n_t, n_c, m, n_rhs, s, st);
#define MM_OLS_GO(T, TIN) \
  ols_dispatch<T, TIN>(logn, variant, y_in, y_out, chunks, n_chunks, spec, ptw, qtw, n_t, n_c, m, n_rhs, s, st)
  if (fp64) return in_f64 ? MM_OLS_GO(double, double) : MM_OLS_GO(double, float);
  return in_f64 ? MM_OLS_GO(float, double) : MM_OLS_GO(float, float);
#undef MM_OLS_GO
}

}  // namespace mm
