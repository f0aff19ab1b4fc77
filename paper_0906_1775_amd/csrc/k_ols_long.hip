// Overlap-save N^-1 with transforms longer than one workgroup's registers and LDS
// (n_f = 2^17 and 2^18: the lengths of the paper's FFT-length rule for n_c = 8192,
// Weighting section, eqs. FFTcomplexity and FFTcomplexityFunction).
//
// The n_f = 2N real window x is z_n = x_n - i x_(n+N) (negacyclic embedding, see
// k_ols_wave.hip), N = N1 x N2, and its shifted transform runs by the four-step
// decomposition, n = N2 n1 + n2, k = k1 + N1 k2:
//   Z[k1 + N1 k2] = sum_n2 W_N2^(n2 k2) [ W_N^(n2 (k1 + 1/4)) sum_n1 z[N2 n1 + n2] W_N1^(n1 (k1 + 1/4)) ],
// in three kernels over a batch of (chunk, RHS) jobs whose N-point intermediates
// stay in device memory (sized so that a batch fits the last-level cache):
//   columns  shifted N1-point transforms of the N2 columns (16 per workgroup, staged through
//            LDS so that every global access covers 16 consecutive points), times
//            W_N^(n2 (k1 + 1/4)), stored as rows Y[k1][n2];
//   rows     N2-point transform of row k1 (one wavefront), conj(F Z), then the N2-point
//            transform of the inverse's first step, times W_N^((k1 + 1/4) n2), in place;
//   output   N1-point transforms of the columns times W_N1^(n1 / 4), and the valid outputs
//            (the real parts y_n and the imaginary parts y_(n+N)) written back.
// The 1/N of the inverse is in the symbol table F / N.
#include <algorithm>

#include "fft.hpp"
#include "mm_internal.h"

namespace mm {

namespace {

// One sub-transform of 2^L points per wavefront: 64 threads x 4 (L = 8, radix-4 passes)
// or x 8 (L = 9, radix-8 passes) points; its per-pass twiddle tables are those of the
// on-chip transform of the same length (launch_pass_twiddles(L, ..., 0)).
template <int L> struct SubShape;
template <> struct SubShape<8> { static constexpr int LOGE = 2; };
template <> struct SubShape<9> { static constexpr int LOGE = 3; };
template <typename T, int L>
using SubFFT = BlockFFT<T, L, 64, SubShape<L>::LOGE, SubShape<L>::LOGE>;

constexpr int kL1 = kLongRowLog;   // columns are 2^8-point transforms
constexpr int kCW = 16;    // columns per workgroup of the column kernels (one per wavefront)

// Table of the four-step transform: W_N^(n2 (k1 + 1/4)) = exp(-2 pi i j / (4N)), j = n2 (4 k1 + 1)
// < 4N, as hi[j / (4 N2)] lo[j mod (4 N2)]: lo[j] = exp(-2 pi i j / (4N)) (j < 4 N2),
// hi[j] = exp(-2 pi i j / N1) (j < N1).
template <typename T, int L1, int L2>
struct LongTables {
  static constexpr int N1 = 1 << L1, N2 = 1 << L2;
  static constexpr int LO = 0, HI = 4 * N2, TOTAL = 4 * N2 + N1;
};

// W_N^(n2 (k1 + 1/4))
template <typename T, int L1, int L2>
__device__ __forceinline__ cx<T> w_n(const cx<T>* __restrict__ tab, int n2, int k1) {
  using LT = LongTables<T, L1, L2>;
  const int j = n2 * (4 * k1 + 1);
  return cmul(tab[LT::HI + (j >> (L2 + 2))], tab[LT::LO + (j & (4 * LT::N2 - 1))]);
}

template <typename T, int L1, int L2>
constexpr int col_lds_bytes() {
  constexpr int a = kCW * SubFFT<T, L1>::LDS_BYTES;
  constexpr int b = kCW * ((1 << L1) + 1) * (int)sizeof(cx<T>);
  constexpr int c = (1 << L1) * (kCW + 1) * (int)sizeof(cx<T>);
  return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

}  // namespace

// Block of the column kernels: the hardware deals blocks to the 8 XCDs in turn, so XCD x takes
// a contiguous run of column groups (their count is a multiple of 16), and neighbouring
// groups, whose 64-byte runs of float32 samples share cache lines, meet in one L2.
__device__ __forceinline__ uint32_t xcd_block() {
  return (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

// The mean of a job's window (window_mean)
template <typename T, typename Tin, int N>
__device__ __forceinline__ T long_mean(const Tin* __restrict__ src, int64_t s0, int64_t lo, int64_t hi) {
  return window_mean<T, 2 * N>(threadIdx.x, [&](int n) { return s0 + n >= lo && s0 + n < hi ? (T)src[s0 + n] : (T)0; });
}

// columns of the forward transform: work[j][k1][n2] = W_N^(n2 (k1 + 1/4)) sum_n1 z[N2 n1 + n2] W_N1^(n1 (k1 + 1/4))
template <typename T, typename Tin, int L1, int L2>
__global__ __launch_bounds__(1024) void k_long_columns(const Tin* __restrict__ yin, cx<T>* __restrict__ work,
                                                       const OlsChunk* __restrict__ chunks, int64_t job0,
                                                       int n_chunks, int64_t n_t, int n_c,
                                                       const CgState* __restrict__ st,
                                                       const cx<T>* __restrict__ ptw1,
                                                       const cx<T>* __restrict__ ltab) {
  using F1 = SubFFT<T, L1>;
  constexpr int N1 = 1 << L1, N2 = 1 << L2, NG = N2 / kCW, TS = N1 + 1, OS = kCW + 1;
  constexpr int64_t N = (int64_t)N1 * N2;
  __shared__ __align__(16) char lds[col_lds_bytes<T, L1, L2>()];
  const uint32_t wg = xcd_block();
  const int64_t jl = wg / NG;
  const int cg = wg % NG;
  const int64_t job = job0 + jl;
  const int rhs = (int)(job / n_chunks);
  if (st && !st[rhs].active) return;   // this RHS has stopped iterating
  const OlsChunk ch = chunks[job - (int64_t)rhs * n_chunks];
  const Tin* __restrict__ src = yin + (int64_t)rhs * n_t;
  const int64_t s0 = ch.out_start - n_c, lo = ch.iv_lo, hi = ch.iv_hi;
  const T mean = long_mean<T, Tin, (int)N>(src, s0, lo, hi);
  cx<T>* tile = reinterpret_cast<cx<T>*>(lds);
  const int tid = threadIdx.x;
  // the workgroup's 16 columns, row by row: 16 consecutive points = two runs of 16 samples
#pragma unroll
  for (int q = 0; q < N1 * kCW / 1024; ++q) {
    const int e = tid + 1024 * q;
    const int c = e % kCW, n1 = e / kCW;
    const int64_t j = s0 + (int64_t)N2 * n1 + cg * kCW + c;
    const T a = (j >= lo && j < hi) ? (T)src[j] : (T)0;
    const T b = (j + N >= lo && j + N < hi) ? (T)src[j + N] : (T)0;
    tile[c * TS + n1] = {a - mean, mean - b};
  }
  __syncthreads();
  const int w = tid >> 6, t = tid & 63;   // wavefront w transforms column cg * 16 + w
  cx<T> v[F1::E];
#pragma unroll
  for (int r = 0; r < F1::E; ++r) v[r] = tile[w * TS + t + 64 * r];
  // (the transform's first exchange begins with a barrier: every column is in registers
  // before any wavefront reuses the tile's LDS)
  F1::template forward<true>(v, lds + w * F1::LDS_BYTES, ptw1, t);
  const int n2 = cg * kCW + w;
#pragma unroll
  for (int r = 0; r < F1::E; ++r) v[r] = cmul(v[r], w_n<T, L1, L2>(ltab, n2, t + 64 * r));
  __syncthreads();
#pragma unroll
  for (int r = 0; r < F1::E; ++r) tile[(t + 64 * r) * OS + w] = v[r];
  __syncthreads();
  cx<T>* __restrict__ dst = work + jl * N;
#pragma unroll
  for (int q = 0; q < N1 * kCW / 1024; ++q) {
    const int e = tid + 1024 * q;
    const int c = e % kCW, k1 = e / kCW;
    dst[(int64_t)k1 * N2 + cg * kCW + c] = tile[k1 * OS + c];
  }
}

// row k1: N2-point transform, symbol, then the first step of the inverse (N2-point
// transform, times W_N^((k1 + 1/4) n2)), in place; one row per wavefront
constexpr int kRowWaves = 1;
template <typename T, int L1, int L2>
__global__ __launch_bounds__(64 * kRowWaves) void k_long_rows(cx<T>* __restrict__ work,
                                                              const OlsChunk* __restrict__ chunks, int64_t job0,
                                                              int n_chunks, const CgState* __restrict__ st,
                                                              const T* __restrict__ spec_rows,
                                                              const cx<T>* __restrict__ ptw2,
                                                              const cx<T>* __restrict__ ltab) {
  using F2 = SubFFT<T, L2>;
  constexpr int N1 = 1 << L1, N2 = 1 << L2, WG = N1 / kRowWaves;
  constexpr int64_t N = (int64_t)N1 * N2;
  __shared__ __align__(16) char lds[kRowWaves * F2::LDS_BYTES];
  const int64_t jl = blockIdx.x / WG;
  const int64_t job = job0 + jl;
  const int rhs = (int)(job / n_chunks);
  if (st && !st[rhs].active) return;   // this RHS has stopped iterating
  const OlsChunk ch = chunks[job - (int64_t)rhs * n_chunks];
  const int w = threadIdx.x >> 6, t = threadIdx.x & 63;
  const int row = (int)(blockIdx.x % WG) * kRowWaves + w;
  cx<T>* __restrict__ base = work + jl * N + (int64_t)row * N2;
  cx<T> v[F2::E];
#pragma unroll
  for (int r = 0; r < F2::E; ++r) v[r] = base[t + 64 * r];
  F2::forward_rev(v, lds + w * F2::LDS_BYTES, ptw2, t);
  // v[r] = Z[row + N1 k2], k2 = t + 64 r; the symbol in row order
  const T* __restrict__ SR = spec_rows + (int64_t)ch.filter * (N + 1) + (int64_t)row * N2;
#pragma unroll
  for (int r = 0; r < F2::E; ++r) {
    const T f = SR[t + 64 * r];
    v[r] = {v[r].re * f, -(v[r].im * f)};
  }
  F2::forward_rev(v, lds + w * F2::LDS_BYTES, ptw2, t);
#pragma unroll
  for (int r = 0; r < F2::E; ++r) base[t + 64 * r] = cmul(v[r], w_n<T, L1, L2>(ltab, t + 64 * r, row));
}

// columns of the inverse: N1-point transforms over k1, times W_N1^(n1 / 4), and the valid outputs
template <typename T, typename Tin, int L1, int L2>
__global__ __launch_bounds__(1024) void k_long_output(const Tin* __restrict__ yin, const cx<T>* __restrict__ work,
                                                      T* __restrict__ yout, const T* __restrict__ spec_rows,
                                                      const OlsChunk* __restrict__ chunks, int64_t job0,
                                                      int n_chunks, int64_t n_t, int n_c, int m,
                                                      const CgState* __restrict__ st,
                                                      const cx<T>* __restrict__ ptw1,
                                                      const cx<T>* __restrict__ qtw) {
  using F1 = SubFFT<T, L1>;
  constexpr int N1 = 1 << L1, N2 = 1 << L2, NG = N2 / kCW, TS = N1 + 1, OS = kCW + 1;
  constexpr int64_t N = (int64_t)N1 * N2;
  __shared__ __align__(16) char lds[col_lds_bytes<T, L1, L2>()];
  const uint32_t wg = xcd_block();
  const int64_t jl = wg / NG;
  const int cg = wg % NG;
  const int64_t job = job0 + jl;
  const int rhs = (int)(job / n_chunks);
  if (st && !st[rhs].active) return;   // this RHS has stopped iterating
  const OlsChunk ch = chunks[job - (int64_t)rhs * n_chunks];
  const int64_t s0 = ch.out_start - n_c, hi = ch.iv_hi;
  const T back = long_mean<T, Tin, (int)N>(yin + (int64_t)rhs * n_t, s0, ch.iv_lo, hi) *
                 spec_rows[(int64_t)ch.filter * (N + 1) + N];   // what the filter makes of the mean
  cx<T>* tile = reinterpret_cast<cx<T>*>(lds);
  const int tid = threadIdx.x;
  const cx<T>* __restrict__ srcw = work + jl * N;
#pragma unroll
  for (int q = 0; q < N1 * kCW / 1024; ++q) {
    const int e = tid + 1024 * q;
    const int c = e % kCW, k1 = e / kCW;
    tile[c * TS + k1] = srcw[(int64_t)k1 * N2 + cg * kCW + c];
  }
  __syncthreads();
  const int w = tid >> 6, t = tid & 63;
  cx<T> v[F1::E];
#pragma unroll
  for (int r = 0; r < F1::E; ++r) v[r] = tile[w * TS + t + 64 * r];
  F1::forward_rev(v, lds + w * F1::LDS_BYTES, ptw1, t);
#pragma unroll
  for (int r = 0; r < F1::E; ++r) v[r] = cmul(v[r], qtw[t + 64 * r]);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < F1::E; ++r) tile[(t + 64 * r) * OS + w] = v[r];   // output n1 = t + 64 r
  __syncthreads();
  T* __restrict__ dst = yout + (int64_t)rhs * n_t;
#pragma unroll
  for (int q = 0; q < N1 * kCW / 1024; ++q) {
    const int e = tid + 1024 * q;
    const int c = e % kCW, n1 = e / kCW;
    const int64_t pos = (int64_t)N2 * n1 + cg * kCW + c;
    const cx<T> z = tile[n1 * OS + c];
    if (pos >= n_c && pos < n_c + m && s0 + pos < hi) dst[s0 + pos] = z.re + back;
    if (pos + N >= n_c && pos + N < n_c + m && s0 + pos + N < hi) dst[s0 + pos + N] = z.im + back;
  }
}

// LongTables of a transform of 2^logn points, from float64 angles
template <typename T, int L1, int L2>
__global__ void k_long_tables(cx<T>* __restrict__ tab) {
  using LT = LongTables<T, L1, L2>;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= LT::TOTAL) return;
  double frac;   // angle / (-2 pi)
  if (e < LT::HI) frac = (double)e / (4.0 * LT::N1 * LT::N2);
  else frac = (double)(e - LT::HI) / (double)LT::N1;
  double sn, cs;
  sincospi(2.0 * frac, &sn, &cs);
  tab[e] = {(T)cs, (T)(-sn)};
}

int ols_long_table_count(int logn) { return 4 * (1 << (logn - kL1)) + (1 << kL1); }

template <typename T, int L2>
static hipError_t long_tables_launch(void* tab, hipStream_t s) {
  using LT = LongTables<T, kL1, L2>;
  hipLaunchKernelGGL((k_long_tables<T, kL1, L2>), dim3((LT::TOTAL + 255) / 256), dim3(256), 0, s, (cx<T>*)tab);
  return hipGetLastError();
}

hipError_t launch_long_tables(int logn, bool fp64, void* tab, hipStream_t s) {
  if (logn == kL1 + 8) return fp64 ? long_tables_launch<double, 8>(tab, s) : long_tables_launch<float, 8>(tab, s);
  if (logn == kL1 + 9) return fp64 ? long_tables_launch<double, 9>(tab, s) : long_tables_launch<float, 9>(tab, s);
  return hipErrorInvalidValue;
}

bool ols_long_exists(int logn) { return logn == kL1 + 8 || logn == kL1 + 9; }

int64_t ols_long_batch(int logn, bool fp64) {
  const int64_t job_bytes = (int64_t(1) << logn) * (fp64 ? 16 : 8);
  return std::max<int64_t>(1, (int64_t(64) << 20) / job_bytes);
}

template <typename T, typename Tin, int L2>
static hipError_t long_launch(const void* y_in, void* y_out, const OlsChunk* chunks, int n_chunks, const void* spec,
                              const void* ptw1, const void* ptw2, const void* qtw, const void* ltab, void* work,
                              int64_t batch, int64_t n_t, int n_c, int m, int n_rhs, hipStream_t s,
                              const CgState* st) {
  constexpr int NG = (1 << L2) / kCW, NP = (1 << kL1) / kRowWaves;
  const int64_t n_jobs = (int64_t)n_chunks * n_rhs;
  for (int64_t j0 = 0; j0 < n_jobs; j0 += batch) {
    const int64_t nb = std::min(batch, n_jobs - j0);
    hipLaunchKernelGGL((k_long_columns<T, Tin, kL1, L2>), dim3((unsigned)(nb * NG)), dim3(1024), 0, s,
                       (const Tin*)y_in, (cx<T>*)work, chunks, j0, n_chunks, n_t, n_c, st, (const cx<T>*)ptw1,
                       (const cx<T>*)ltab);
    hipLaunchKernelGGL((k_long_rows<T, kL1, L2>), dim3((unsigned)(nb * NP)), dim3(64 * kRowWaves), 0, s, (cx<T>*)work,
                       chunks, j0, n_chunks, st, (const T*)spec, (const cx<T>*)ptw2, (const cx<T>*)ltab);
    hipLaunchKernelGGL((k_long_output<T, Tin, kL1, L2>), dim3((unsigned)(nb * NG)), dim3(1024), 0, s,
                       (const Tin*)y_in, (const cx<T>*)work, (T*)y_out, (const T*)spec, chunks, j0, n_chunks, n_t, n_c, m, st, (const cx<T>*)ptw1,
                       (const cx<T>*)qtw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, typename Tin>
static hipError_t long_dispatch(int logn, const void* y_in, void* y_out, const OlsChunk* chunks, int n_chunks,
                                const void* spec, const void* ptw1, const void* ptw2, const void* qtw,
                                const void* ltab, void* work, int64_t batch, int64_t n_t, int n_c, int m, int n_rhs,
                                hipStream_t s, const CgState* st) {
  if (logn == kL1 + 8)
    return long_launch<T, Tin, 8>(y_in, y_out, chunks, n_chunks, spec, ptw1, ptw2, qtw, ltab, work, batch, n_t, n_c,
                                  m, n_rhs, s, st);
  if (logn == kL1 + 9)
    return long_launch<T, Tin, 9>(y_in, y_out, chunks, n_chunks, spec, ptw1, ptw2, qtw, ltab, work, batch, n_t, n_c,
                                  m, n_rhs, s, st);
  return hipErrorInvalidValue;
}

hipError_t launch_ols_long(bool fp64, bool in_f64, int logn, const void* y_in, void* y_out, const OlsChunk* chunks,
                           int n_chunks, const void* spec_rows, const void* ptw1, const void* ptw2, const void* qtw,
                           const void* ltab, void* work, int64_t batch, int64_t n_t, int n_c, int m, int n_rhs,
                           hipStream_t s, const CgState* st) {
  if (n_chunks == 0 || n_rhs == 0) return hipSuccess;
  if (batch < 1) return hipErrorInvalidValue;
  if (fp64)
    return in_f64 ? long_dispatch<double, double>(logn, y_in, y_out, chunks, n_chunks, spec_rows, ptw1, ptw2, qtw,
                                                  ltab, work, batch, n_t, n_c, m, n_rhs, s, st)
                  : long_dispatch<double, float>(logn, y_in, y_out, chunks, n_chunks, spec_rows, ptw1, ptw2, qtw,
                                                 ltab, work, batch, n_t, n_c, m, n_rhs, s, st);
  return in_f64 ? long_dispatch<float, double>(logn, y_in, y_out, chunks, n_chunks, spec_rows, ptw1, ptw2, qtw, ltab,
                                               work, batch, n_t, n_c, m, n_rhs, s, st)
                : long_dispatch<float, float>(logn, y_in, y_out, chunks, n_chunks, spec_rows, ptw1, ptw2, qtw, ltab,
                                              work, batch, n_t, n_c, m, n_rhs, s, st);
}

}  // namespace mm
