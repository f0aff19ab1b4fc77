// Template columns B of the extended pointing [P B] ("Using MADmap" section
// of the MADmap paper, eqs. eDSN1 and PmatExt), and the white-noise weighting
// used when n_c = 1.
//
// One-hot templates (synchronous bins, destriping offsets) are pointing
// matrices of their own with one unit weight per row: the plan builds them
// with the pixel machinery (sort, observed compaction, sliced scatter) and
// only the gather into an existing TOD needs a kernel here.
//
// The half-wave-plate block (eq. HWPmat) has 32 dense columns per segment,
// evaluated on the fly from the polarizer angle w_t: for k = 1..8,
// cos(k w), tau cos(k w), sin(k w), tau sin(k w), with tau the sample index
// centred on the segment and scaled to (-1, 1).  cos(k w) and sin(k w) come
// from one sincos and the angle-addition recurrence, in float64.  Samples are
// cut into tiles of at most kTileSamples samples inside one segment; the scatter
// writes one partial sum per tile and column, and a second kernel adds the
// tiles of each segment in order (no atomics, fixed summation order).
#include <algorithm>

#include "mm_internal.h"

namespace mm {

static dim3 grid_for(int64_t n) {
  int64_t nb = (n + 255) / 256;
  if (nb > 65536) nb = 65536;
  if (nb < 1) nb = 1;
  return dim3((unsigned)nb);
}

// ---------------------------------------------------------------- one-hot gather
template <typename Ty>
__global__ void k_onehot_gather(const int32_t* __restrict__ obs_idx, const double* __restrict__ p,
                                int64_t vs, int64_t off, Ty* __restrict__ y, int64_t n_t, int n_rhs,
                                const CgState* __restrict__ st) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_t; t += stride) {
    const int32_t o = obs_idx[t];
    if (o < 0) continue;
    for (int r = 0; r < n_rhs; ++r) {
      if (st && !st[r].active) continue;
      const int64_t i = (int64_t)r * n_t + t;
      y[i] = (Ty)((double)y[i] + p[(int64_t)r * vs + off + o]);
    }
  }
}

hipError_t launch_onehot_gather(bool y_f64, const int32_t* obs_idx, const double* p, int64_t vs, int64_t off,
                                void* y, int64_t n_t, int n_rhs, hipStream_t s, const CgState* st) {
  if (n_t == 0) return hipSuccess;
  if (y_f64) hipLaunchKernelGGL(k_onehot_gather<double>, grid_for(n_t), dim3(256), 0, s, obs_idx, p, vs, off, (double*)y, n_t, n_rhs, st);
  else hipLaunchKernelGGL(k_onehot_gather<float>, grid_for(n_t), dim3(256), 0, s, obs_idx, p, vs, off, (float*)y, n_t, n_rhs, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------- HWP block
// 2/pi, 3 zero bits before the 253 bits that follow the point
__device__ const unsigned long long kTwoOverPi[4] = {0x145f306dc9c882a5ull, 0x3f84eafa3ea69bb8ull, 0x1b6c52b327887208ull, 0x3fca2c757bd778acull};

// sin and cos of a float32 angle in float64 (errors below 2e-16): the angle less n pi/2, then
// the Taylor polynomials on [-pi/4, pi/4] to x^17 and x^16 (next terms below 1e-17).  Up to
// 2^22 the remainder takes two steps with pi/2 as a pair of float64 (n times the first is
// exact inside its fma); beyond, w = m 2^e with an integer m, and m 2^e 2/pi mod 4 needs
// only the 128 bits of 2/pi from the weight 2 / 2^e on (Payne and Hanek's reduction).  The
// library's sincos took half again the registers in the kernels below.
__device__ __forceinline__ void sincos_f32(float w, double* sn, double* cs) {
  double r;
  int k;
  if (fabsf(w) <= 4194304.0f) {
    const double n = rint((double)w * 0.6366197723675814);
    r = fma(-n, 1.5707963267948966, (double)w);    // pi/2 rounded to float64
    r = fma(-n, 6.123233995736766e-17, r);            // and what that left out
    k = (int)n;
  } else {
    const uint32_t bits = __float_as_uint(w);
    const int ex = (int)((bits >> 23) & 255);
    const int at = ex == 255 ? 0 : ex - 149;                        // e + 1, in 0 .. 105
    const unsigned long long m = (bits & 0x7fffff) | 0x800000;
    const int i = at >> 6, sh = at & 63;
    const unsigned long long a = kTwoOverPi[i], b = kTwoOverPi[i + 1], c = i + 2 < 4 ? kTwoOverPi[i + 2] : 0;
    const unsigned long long hi = sh ? a << sh | b >> (64 - sh) : a, lo = sh ? b << sh | c >> (64 - sh) : b;
    const unsigned long long q = hi * m + __umul64hi(lo, m);        // 2^62 to a quarter turn
    const long long f = (long long)(q << 2);                        // remainder as a signed part of 2^64
    k = (int)(q >> 62) + (f < 0 ? 1 : 0);
    r = (double)f * (1.5707963267948966 / 18446744073709551616.0);
    if (bits >> 31) k = -k, r = -r;
    if (ex == 255) r = (double)(w - w);                             // infinity and NaN
  }
  const double z = r * r;
  double p = fma(z, 1.0 / 355687428096000.0, -1.0 / 1307674368000.0);
  p = fma(z, p, 1.0 / 6227020800.0);
  p = fma(z, p, -1.0 / 39916800.0);
  p = fma(z, p, 1.0 / 362880.0);
  p = fma(z, p, -1.0 / 5040.0);
  p = fma(z, p, 1.0 / 120.0);
  p = fma(z, p, -1.0 / 6.0);
  const double s = fma(r * z, p, r);
  double q = fma(z, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);
  q = fma(z, q, 1.0 / 479001600.0);
  q = fma(z, q, -1.0 / 3628800.0);
  q = fma(z, q, 1.0 / 40320.0);
  q = fma(z, q, -1.0 / 720.0);
  q = fma(z, q, 1.0 / 24.0);
  q = fma(z, q, -0.5);
  const double c = fma(z, q, 1.0);
  const double a = k & 1 ? c : s, b = k & 1 ? s : c;
  *sn = k & 2 ? -a : a;
  *cs = (k + 1) & 2 ? -b : b;
}

__device__ __forceinline__ void hwp_harmonics(float w, double* c, double* sn) {
  double s1, c1;
  sincos_f32(w, &s1, &c1);
  c[0] = c1;
  sn[0] = s1;
#pragma unroll
  for (int k = 1; k < kHwpHarmonics; ++k) {
    c[k] = c[k - 1] * c1 - sn[k - 1] * s1;
    sn[k] = sn[k - 1] * c1 + c[k - 1] * s1;
  }
}

__device__ __forceinline__ double hwp_tau(int64_t t, int64_t s0, double L, double inv_L) {
  return (2.0 * (double)(t - s0) - (L - 1.0)) * inv_L;
}

// Samples whose angle and TOD value a thread of the two kernels below has in flight: a plan
// of 2^22 samples has 4 wavefronts on a SIMD, too few to cover the loads one by one.
constexpr int kHwpAhead = 4;

// y[r][t] += sum_i C[t][i] a[r][seg(t)][i] over the tiles.  Bound by the float64 arithmetic
// (about 110 instructions a sample).  The 32 amplitudes of a row are the same for the whole
// block and are read with scalar loads.  ONE: a single right-hand side, its values fetched ahead.
template <typename Ty, bool ONE>
__global__ __launch_bounds__(256) void k_hwp_gather(const SampleTile* __restrict__ tiles,
                                                    const int64_t* __restrict__ seg_start,
                                                    const float* __restrict__ omega, const double* __restrict__ p,
                                                    int64_t vs, int64_t off, Ty* __restrict__ y, int64_t n_t,
                                                    int n_rhs, const CgState* __restrict__ st) {
  if (ONE && st && !st[0].active) return;
  const SampleTile T = tiles[blockIdx.x];
  const int64_t s0 = seg_start[T.id];
  const double L = (double)(seg_start[T.id + 1] - s0), inv_L = 1.0 / L;
  const double* __restrict__ seg = p + off + (int64_t)T.id * kHwpColumns;
  for (int64_t b0 = T.t0 + threadIdx.x; b0 < T.t1; b0 += kHwpAhead * 256) {
    float w[kHwpAhead];
    Ty y1[kHwpAhead];
#pragma unroll
    for (int j = 0; j < kHwpAhead; ++j) {
      const int64_t t = b0 + j * 256 < T.t1 ? b0 + j * 256 : b0;
      w[j] = omega[t];
      if (ONE) y1[j] = y[t];
    }
#pragma unroll 1
    for (int j = 0; j < kHwpAhead; ++j) {
      const int64_t t = b0 + j * 256;
      if (t >= T.t1) break;
      double c[kHwpHarmonics], sn[kHwpHarmonics];
      hwp_harmonics(w[0], c, sn);
      const double tau = hwp_tau(t, s0, L, inv_L);
      for (int r = 0; r < (ONE ? 1 : n_rhs); ++r) {
        if (!ONE && st && !st[r].active) continue;
        const double* __restrict__ ar = seg + (int64_t)r * vs;
        const int64_t i = (int64_t)r * n_t + t;
        const Ty y0 = ONE ? y1[0] : y[i];
        double v = 0.0, u = 0.0;
#pragma unroll
        for (int k = 0; k < kHwpHarmonics; ++k) {
          v = fma(ar[k], c[k], fma(ar[16 + k], sn[k], v));
          u = fma(ar[8 + k], c[k], fma(ar[24 + k], sn[k], u));
        }
        y[i] = (Ty)((double)y0 + fma(tau, u, v));
      }
#pragma unroll
      for (int i = 0; i + 1 < kHwpAhead; ++i) w[i] = w[i + 1], y1[i] = y1[i + 1];
    }
  }
}

hipError_t launch_hwp_gather(bool y_f64, const SampleTile* tiles, int n_tiles, const int64_t* seg_start,
                             const float* omega, const double* p, int64_t vs, int64_t off, void* y, int64_t n_t,
                             int n_rhs, hipStream_t s, const CgState* st) {
  if (n_tiles == 0) return hipSuccess;
  if (n_rhs > kMaxRhs) return hipErrorInvalidValue;
#define MM_HG(TY, ONE) hipLaunchKernelGGL((k_hwp_gather<TY, ONE>), dim3(n_tiles), dim3(256), 0, s, tiles, seg_start, \
                                          omega, p, vs, off, (TY*)y, n_t, n_rhs, st)
  if (y_f64) { if (n_rhs == 1) MM_HG(double, true); else MM_HG(double, false); }
  else { if (n_rhs == 1) MM_HG(float, true); else MM_HG(float, false); }
#undef MM_HG
  return hipGetLastError();
}

// white-noise weight f_b(0) of sample t (interval by binary search; plan time only)
__device__ __forceinline__ double white_weight(int64_t t, const int64_t* __restrict__ iv_start, int n_iv,
                                               const int32_t* __restrict__ iv_filter,
                                               const double* __restrict__ lags, int n_c) {
  int lo = 0, hi = n_iv;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (iv_start[mid] <= t) lo = mid; else hi = mid;
  }
  return lags[(int64_t)iv_filter[lo] * n_c];
}

// partial[tile][r][i] = sum over the tile of C[t][i] y[r][t]            (kSum)
// partial[tile][0][i] = sum over the tile of C[t][i]^2 w(t)             (kNoise: w = f_b(0); kUnit: w = 1)
enum class HwpSum { kSum, kNoise, kUnit };
template <typename Ty, HwpSum MODE>
__global__ __launch_bounds__(256, 4) void k_hwp_scatter(const SampleTile* __restrict__ tiles,
                                                     const int64_t* __restrict__ seg_start,
                                                     const float* __restrict__ omega, const Ty* __restrict__ y,
                                                     int64_t n_t, int n_rhs, double* __restrict__ partial,
                                                     const int64_t* __restrict__ iv_start, int n_iv,
                                                     const int32_t* __restrict__ iv_filter,
                                                     const double* __restrict__ lags, int n_c,
                                                     const CgState* __restrict__ st) {
  __shared__ double red[256 / 64][kHwpColumns];
  const SampleTile T = tiles[blockIdx.x];
  const int64_t s0 = seg_start[T.id];
  const double L = (double)(seg_start[T.id + 1] - s0), inv_L = 1.0 / L;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int R = MODE == HwpSum::kSum ? n_rhs : 1;
  for (int r = 0; r < R; ++r) {
    if (st && !st[r].active) continue;     // uniform over the block
    const Ty* __restrict__ yr = y + (int64_t)r * n_t;
    double acc[kHwpColumns];
#pragma unroll
    for (int i = 0; i < kHwpColumns; ++i) acc[i] = 0.0;
    for (int64_t b0 = T.t0 + threadIdx.x; b0 < T.t1; b0 += kHwpAhead * 256) {
      float w[kHwpAhead];
      Ty y1[kHwpAhead];
#pragma unroll
      for (int j = 0; j < kHwpAhead; ++j) {
        const int64_t t = b0 + j * 256 < T.t1 ? b0 + j * 256 : b0;
        w[j] = omega[t];
        if (MODE == HwpSum::kSum) y1[j] = yr[t];
      }
#pragma unroll 1
      for (int j = 0; j < kHwpAhead; ++j) {
        const int64_t t = b0 + j * 256;
        if (t >= T.t1) break;
        double s1, c1;
        sincos_f32(w[0], &s1, &c1);
        const double tau = hwp_tau(t, s0, L, inv_L);
        double v = 1.0;
        if (MODE == HwpSum::kSum) v = (double)y1[0];
        if (MODE == HwpSum::kNoise) v = white_weight(t, iv_start, n_iv, iv_filter, lags, n_c);
        const double tv = MODE == HwpSum::kSum ? tau * v : tau * tau * v;
        double c = c1, sn = s1;
#pragma unroll
        for (int k = 0; k < kHwpHarmonics; ++k) {
          const double a = MODE == HwpSum::kSum ? c : c * c, b = MODE == HwpSum::kSum ? sn : sn * sn;
          acc[k] += a * v;
          acc[8 + k] += a * tv;
          acc[16 + k] += b * v;
          acc[24 + k] += b * tv;
          const double c2 = c * c1 - sn * s1;
          sn = sn * c1 + c * s1;
          c = c2;
        }
#pragma unroll
        for (int i = 0; i + 1 < kHwpAhead; ++i) w[i] = w[i + 1], y1[i] = y1[i + 1];
      }
    }
    // 32 sums over 64 lanes: at each level a lane hands half of its columns to a partner and
    // adds the partner's part of the other half, so lanes 2 i and 2 i + 1 end with column i
    // (32 exchanges instead of 6 for every column)
#pragma unroll
    for (int h = kHwpColumns / 2; h >= 1; h >>= 1) {
      const bool up = lane & (2 * h);
#pragma unroll
      for (int i = 0; i < h; ++i) {
        const double mine = up ? acc[h + i] : acc[i], theirs = up ? acc[i] : acc[h + i];
        acc[i] = mine + __shfl_xor(theirs, 2 * h, 64);
      }
    }
    acc[0] += __shfl_xor(acc[0], 1, 64);
    if ((lane & 1) == 0) red[wv][lane >> 1] = acc[0];
    __syncthreads();
    if (threadIdx.x < kHwpColumns) {
      double v = 0.0;
      for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v += red[w][threadIdx.x];
      partial[((int64_t)blockIdx.x * R + r) * kHwpColumns + threadIdx.x] = v;
    }
    __syncthreads();
  }
}

// q[r][off + 32 g + i] = sum over the tiles of segment g of partial[tile][r][i], in an order
// that TL fixes; with p, also pq_part[r * pq_stride + pq_slot + block] = sum of p q over the
// block.  32 groups of 32 threads (one per column): TL groups share a segment, each adding every
// TL-th tile, so a few long segments fill a block as well as many short ones (4 segments of 256
// tiles, one thread per column: 62 us, every tile a load behind the last).
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void k_hwp_reduce(const double* __restrict__ partial,
                                                    const int32_t* __restrict__ seg_tile, int n_seg, int tl, int n_rhs,
                                                    double* __restrict__ q, int64_t vs, int64_t off,
                                                    const double* __restrict__ p, double* __restrict__ pq_part,
                                                    int pq_stride, int pq_slot, const CgState* __restrict__ st) {
  constexpr int NG = kReduceThreads / kHwpColumns;
  __shared__ double part[NG][kHwpColumns];
  __shared__ double sh[kReduceThreads / 64];
  const int r = blockIdx.y;
  if (st && !st[r].active) return;
  const int i = threadIdx.x % kHwpColumns, grp = threadIdx.x / kHwpColumns;
  const int spb = NG / tl, sub = grp % tl;         // segments of a block and step
  double pq = 0.0;
  for (int g0 = blockIdx.x * spb; g0 < n_seg; g0 += gridDim.x * spb) {
    const int g = g0 + grp / tl;
    double v = 0.0;
    if (g < n_seg) {
      const int t1 = seg_tile[g + 1];
#pragma unroll 8
      for (int t = seg_tile[g] + sub; t < t1; t += tl) v += partial[((int64_t)t * n_rhs + r) * kHwpColumns + i];
    }
    part[grp][i] = v;
    __syncthreads();
    if (sub == 0 && g < n_seg) {
      for (int k = 1; k < tl; ++k) v += part[grp + k][i];
      const int64_t e = (int64_t)r * vs + off + (int64_t)g * kHwpColumns + i;
      q[e] = v;
      if (p) pq += p[e] * v;
    }
    __syncthreads();
  }
  if (p) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) pq += __shfl_xor(pq, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = pq;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int w = 0; w < kReduceThreads / 64; ++w) s += sh[w];
      pq_part[(int64_t)r * pq_stride + pq_slot + blockIdx.x] = s;
    }
  }
}

// thread groups per segment: a power of two near a quarter of the mean number of tiles
static int hwp_groups(int n_tiles, int n_seg) {
  int tl = 1;
  while (tl < kReduceThreads / kHwpColumns && (int64_t)tl * 4 * n_seg < n_tiles) tl *= 2;
  return tl;
}

int hwp_reduce_blocks(int n_tiles, int n_seg) {
  const int spb = kReduceThreads / kHwpColumns / hwp_groups(n_tiles, n_seg);
  return std::max(1, std::min((n_seg + spb - 1) / spb, kHwpReduceBlocks));
}

hipError_t launch_hwp_scatter(bool y_f64, const SampleTile* tiles, int n_tiles, const int32_t* seg_tile, int n_seg,
                              const int64_t* seg_start, const float* omega, const void* y, int64_t n_t, int n_rhs,
                              double* partial, double* q, int64_t vs, int64_t off, const double* p,
                              double* pq_part, int pq_stride, int pq_slot, hipStream_t s, const CgState* st) {
  if (n_seg == 0) return hipSuccess;
  if (n_tiles > 0) {
    if (y_f64)
      hipLaunchKernelGGL((k_hwp_scatter<double, HwpSum::kSum>), dim3(n_tiles), dim3(256), 0, s, tiles, seg_start, omega,
                         (const double*)y, n_t, n_rhs, partial, nullptr, 0, nullptr, nullptr, 1, st);
    else
      hipLaunchKernelGGL((k_hwp_scatter<float, HwpSum::kSum>), dim3(n_tiles), dim3(256), 0, s, tiles, seg_start, omega,
                         (const float*)y, n_t, n_rhs, partial, nullptr, 0, nullptr, nullptr, 1, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_hwp_reduce, dim3(hwp_reduce_blocks(n_tiles, n_seg), n_rhs), dim3(kReduceThreads), 0, s, partial,
                     seg_tile, n_seg, hwp_groups(n_tiles, n_seg), n_rhs, q, vs, off, p, pq_part, pq_stride, pq_slot, st);
  return hipGetLastError();
}

// diag[32 g + i] = sum over segment g of C[t][i]^2 w(t) (w = f_b(0) for kind 0, 1 for kind 1)
hipError_t launch_hwp_diag(int kind, const SampleTile* tiles, int n_tiles, const int32_t* seg_tile, int n_seg,
                           const int64_t* seg_start, const float* omega, const int64_t* iv_start, int n_iv,
                           const int32_t* iv_filter, const double* lags, int n_c, double* partial,
                           double* diag, hipStream_t s) {
  if (n_seg == 0) return hipSuccess;
  if (n_tiles > 0) {
#define MM_HD(MODE) hipLaunchKernelGGL((k_hwp_scatter<float, MODE>), dim3(n_tiles), dim3(256), 0, s, tiles, seg_start, \
                                       omega, (const float*)nullptr, (int64_t)0, 1, partial, iv_start, n_iv,          \
                                       iv_filter, lags, n_c, (const CgState*)nullptr)
    if (kind == 0) MM_HD(HwpSum::kNoise);
    else MM_HD(HwpSum::kUnit);
#undef MM_HD
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_hwp_reduce, dim3(hwp_reduce_blocks(n_tiles, n_seg), 1), dim3(kReduceThreads), 0, s, partial,
                     seg_tile, n_seg, hwp_groups(n_tiles, n_seg), 1, diag, (int64_t)0, (int64_t)0,
                     (const double*)nullptr, (double*)nullptr, 0, 0, (const CgState*)nullptr);
  return hipGetLastError();
}

// ---------------------------------------------------------------- diagonal helpers
// out[j] = 1 / d[j] where d[j] > 0, else 0
__global__ void k_invert_diag(const double* __restrict__ d, double* __restrict__ out, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride)
    out[j] = d[j] > 0.0 ? 1.0 / d[j] : 0.0;
}

hipError_t launch_invert_diag(const double* d, double* out, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_invert_diag, grid_for(n), dim3(256), 0, s, d, out, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------- white noise
// y_out[r][t] = f_b(0) y_in[r][t] over tiles that each lie inside one interval
template <typename Ti, typename To>
__global__ __launch_bounds__(256) void k_white(const SampleTile* __restrict__ tiles, const int32_t* __restrict__ iv_filter,
                                               const double* __restrict__ lags, int n_c, const Ti* __restrict__ y_in,
                                               To* __restrict__ y_out, int64_t n_t, const CgState* __restrict__ st) {
  const SampleTile T = tiles[blockIdx.x];
  const int r = blockIdx.y;
  if (st && !st[r].active) return;
  const double f0 = lags[(int64_t)iv_filter[T.id] * n_c];
  const Ti* yi = y_in + (int64_t)r * n_t;
  To* yo = y_out + (int64_t)r * n_t;
  for (int64_t t = T.t0 + threadIdx.x; t < T.t1; t += blockDim.x) yo[t] = (To)(f0 * (double)yi[t]);
}

hipError_t launch_white(bool out_f64, bool in_f64, const SampleTile* tiles, int n_tiles, const int32_t* iv_filter,
                        const double* lags, int n_c, const void* y_in, void* y_out, int64_t n_t, int n_rhs,
                        hipStream_t s, const CgState* st) {
  if (n_tiles == 0) return hipSuccess;
  const dim3 g(n_tiles, n_rhs), b(256);
  if (in_f64 && out_f64) hipLaunchKernelGGL((k_white<double, double>), g, b, 0, s, tiles, iv_filter, lags, n_c, (const double*)y_in, (double*)y_out, n_t, st);
  else if (in_f64) hipLaunchKernelGGL((k_white<double, float>), g, b, 0, s, tiles, iv_filter, lags, n_c, (const double*)y_in, (float*)y_out, n_t, st);
  else if (out_f64) hipLaunchKernelGGL((k_white<float, double>), g, b, 0, s, tiles, iv_filter, lags, n_c, (const float*)y_in, (double*)y_out, n_t, st);
  else hipLaunchKernelGGL((k_white<float, float>), g, b, 0, s, tiles, iv_filter, lags, n_c, (const float*)y_in, (float*)y_out, n_t, st);
  return hipGetLastError();
}

}  // namespace mm
