// Overlap-save N^-1 with transforms of N = 1024 NO complex points whose inner stages stay
// inside one wavefront (NO = 1 .. 32; the paper's transform is the chunked circulant
// embedding of its Weighting section).
//
// Embedding.  A band of half-width n_c is applied exactly, away from the window's ends, by
// any cyclic extension of the window: also by the negacyclic one (t^(2N) = -1 instead of
// 1).  A real window x of 2N samples modulo t^(2N) + 1 is the N complex points
//   z_n = x_n - i x_(n + N)   (t^N = -i),
// so one shifted transform
//   Z_k = sum_n z_n exp(-2 pi i n (k + 1/4) / N)
// holds its whole spectrum, a symmetric band multiplies it by the real symbol
//   F_k = f(0) + 2 sum_tau f(tau) cos(2 pi (k + 1/4) tau / N),
// and no real-to-complex pairing of Z_k with Z_(N-k) is needed between the forward and the
// inverse transform: every point meets only its own symbol value, in the register it is in.
// (The pairing it replaces cost a workgroup exchange, two barriers, 14 operations per point
// and the packing twiddles.)  The inverse is y_n + i y_(n + N) =
// sum_k conj(F_k Z_k) exp(-2 pi i n (k + 1/4) / N) (the table holds F_k / N).
//
// Transform.  n = g + 1024 n_o (g = l + 64 j, l = m + 16 h) and k = k_o + NO (k1 + 16 c1 +
// 64 c2).  The inner stages run by decimation in time with the twiddles inside the
// butterflies (a + w b, a - w b), so that no separate twiddle multiplications remain there.
// A shift of the frequency passes down every level of a decimation in time unchanged, so
// the 1/4 costs nothing in the forward direction, and each stage's leftover twiddle is a
// shift of the next:
//   forward   outer  NO points over n_o           (shift 1/4, constants)        -> k_o
//             workgroup exchange: wavefront w takes row k_o = w (NO = 32: and w + 16)
//             16 points over j, shift s1 = (k_o + 1/4) / NO                     -> k1
//             private exchange, 4 points over h, shift s2 = (k1 + s1) / 16      -> c1
//             private exchange, 16 points over m, shift s3 = (c1 + s2) / 4      -> c2
//   symbol    lane mu = k1 + 16 c1, register c2
//   inverse   16 points over c2 (no shift)                                      -> m
//             private exchange, 4 points over c1, shift m / 16                  -> h
//             private exchange, 16 points over k1, shift l / 64                 -> j
//             twiddle exp(-2 pi i g (k_o + 1/4) / N), workgroup exchange, NO points over
//             k_o (the transpose of the first stage), stores.
// Private exchanges go through the wavefront's own LDS row and need no barrier, so the
// wavefronts of a workgroup drift apart and one's exchanges overlap another's arithmetic.
// In float64 every exchange moves the real parts, then the imaginary parts, through the
// same LDS space.
#include <algorithm>
#include <type_traits>

#include "fft.hpp"
#include "mm_internal.h"
#include "sky.hpp"

namespace mm {

namespace {

constexpr int kWRow = 1088;   // LDS row stride in 8-byte slots (1024 + 64 padding for the second private exchange)

// NO rows of 1024 points; a thread holds C columns of NO points in the outer stages, RPW
// rows of 16 points in the inner ones.
template <int NO, int RPW_>
struct WaveShape {
  static constexpr int N = 1024 * NO;
  static constexpr int RPW = RPW_;               // rows per wavefront
  static constexpr int NW = NO / RPW;            // wavefronts
  static constexpr int NT = 64 * NW;
  static constexpr int E = 16 * RPW;
  static constexpr int C = E / NO;
  static constexpr int LDS_SLOTS = NW * kWRow;
  static constexpr int LOGNO = NO == 1 ? 0 : NO == 2 ? 1 : NO == 4 ? 2 : NO == 8 ? 3 : NO == 16 ? 4 : 5;
  static_assert(NO == 1 << LOGNO && NW * RPW == NO && NW <= 16 && C * NO == E, "shape");
};

// Twiddle tables (complex entries).  A decimation-in-time stage of 2^s points with shift
// sigma needs exp(-2 pi i (j + sigma) / len) for len = 2, 4, .., 2^s, j < max(1, len / 4) (the
// other quarter is -i times these): eight values for a 16-point stage, at 0 for len = 2, else at
// len / 4 + j.  All of them are rounded once, in the tables: as products of the j = 0 ones with
// constants they cost 4 to 8 % of the filter's error.
template <int NO>
struct WaveTables {
  static constexpr int F1 = 0;                      // [NO][8]: sigma = s1, j < max(1, len / 4)
  static constexpr int F2 = F1 + NO * 8;            // [NO][16 k1][2]: sigma = s2
  static constexpr int F3 = F2 + NO * 32;           // [NO][64 mu][8]: sigma = s3
  static constexpr int I2 = F3 + NO * 512;          // [16 m][2]: sigma = m / 16
  static constexpr int I3 = I2 + 32;                // [64 l][8]: sigma = l / 64
  static constexpr int I4 = I3 + 512;               // [NO k_o][1024 g]: exp(-2 pi i g (k_o + 1/4) / N)
  static constexpr int TOTAL = I4 + NO * 1024;
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// cos(2 pi k / 128), k in [0, 32] (correctly rounded decimal expansions)
__host__ __device__ constexpr double cos128_quarter(int k) {
  constexpr double c[33] = {
      1.0, 0.99879545620517239271477160, 0.99518472667219688624483695, 0.98917650996478097345167373,
      0.98078528040323044912618223, 0.97003125319454399260398420, 0.95694033573220886493579788,
      0.94154406518302077841250940, 0.92387953251128675612818318, 0.90398929312344333158620029,
      0.88192126434835502971275686, 0.85772861000027206990226998, 0.83146961230254523707878837,
      0.80320753148064490980667651, 0.77301045336273696081090660, 0.74095112535495909117561689,
      0.70710678118654752440084436, 0.67155895484701840062537685, 0.63439328416364549821517161,
      0.59569930449243334346703652, 0.55557023301960222474283081, 0.51410274419322172659369383,
      0.47139673682599764855638762, 0.42755509343028209432096685, 0.38268343236508977172845998,
      0.33688985339222005068925321, 0.29028467725446236763619237, 0.24298017990326388994827416,
      0.19509032201612826784828486, 0.14673047445536175165885012, 0.09801714032956060199419556,
      0.04906767432741801425495497, 0.0};
  return c[k];
}

// exp(-2 pi i k / 128), a compile-time constant after unrolling
template <typename T>
__device__ __forceinline__ constexpr cx<T> unit128(int k) {
  const int q = (k >> 5) & 3, f = k & 31;   // quarter turns, rest
  const T c = (T)cos128_quarter(f), s = (T)cos128_quarter(32 - f);
  return q == 0 ? cx<T>{c, -s} : q == 1 ? cx<T>{-s, -c} : q == 2 ? cx<T>{-c, s} : cx<T>{s, c};
}

// a + w b and a - w b by fused multiply-adds
template <typename T>
__device__ __forceinline__ cx<T> madd(cx<T> a, cx<T> w, cx<T> b) {
  return {fma(w.re, b.re, fma(-w.im, b.im, a.re)), fma(w.re, b.im, fma(w.im, b.re, a.im))};
}
template <typename T>
__device__ __forceinline__ cx<T> msub(cx<T> a, cx<T> w, cx<T> b) {
  return {fma(-w.re, b.re, fma(w.im, b.im, a.re)), fma(-w.re, b.im, fma(-w.im, b.re, a.im))};
}

// 4-point DFT of (a, w1 b, w2 c, w3 d), natural order out
template <typename T>
__device__ __forceinline__ void bfly4(cx<T>& a, cx<T>& b, cx<T>& c, cx<T>& d, cx<T> w1, cx<T> w2, cx<T> w3) {
  const cx<T> t0 = madd(a, w2, c), t1 = msub(a, w2, c);
  const cx<T> u = cmul(b, w1);
  const cx<T> t2 = madd(u, w3, d), t3 = msub(u, w3, d);
  a = cadd(t0, t2);
  c = csub(t0, t2);
  b = {t1.re + t3.im, t1.im - t3.re};   // t1 - i t3
  d = {t1.re - t3.im, t1.im + t3.re};
}

// Decimation-in-time transform of R = 2^LOGR <= 16 points in registers, natural order in and
// out: X[k] = sum_n v[n] exp(-2 pi i n (k + sigma) / R), by radix-2 butterflies
// (a + w b, a - w b); tw(len, j) = exp(-2 pi i (j + sigma) / len), j < max(1, len / 4).
// SUM6: six operations per butterfly, the difference as 2 a - (a + w b), which carries the
// sum's rounding along; else eight.
template <typename T, int LOGR, bool SUM6, typename Tw>
__device__ __forceinline__ void dit(cx<T>* v, Tw tw) {
  constexpr int R = 1 << LOGR;
  cx<T> x[R];
#pragma unroll
  for (int k = 0; k < R; ++k) x[k] = v[bitrev(k, LOGR)];
#pragma unroll
  for (int s = 1; s <= LOGR; ++s) {
    const int len = 1 << s, half = len >> 1, q = len >> 2;
#pragma unroll
    for (int j = 0; j < (s == 1 ? 1 : q); ++j) {
      const cx<T> u = tw(len, j);
#pragma unroll
      for (int h = 0; h < (s == 1 ? 1 : 2); ++h) {   // j, and a quarter of len further: -i times the twiddle
        const cx<T> wj = h ? cx<T>{u.im, -u.re} : u;
#pragma unroll
        for (int k = j + h * q; k < R; k += len) {
          const cx<T> sum = madd(x[k], wj, x[k + half]);
          x[k + half] = SUM6 ? cx<T>{fma((T)2, x[k].re, -sum.re), fma((T)2, x[k].im, -sum.im)}
                             : msub(x[k], wj, x[k + half]);
          x[k] = sum;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = x[k];
}

// The same for R <= 32, sigma = 1/4 and compile-time twiddles, in radix-4 levels after a
// radix-2 one when LOGR is odd (28 operations per radix-4 butterfly, fewer roundings)
template <typename T, int LOGR>
__device__ __forceinline__ void dit_quarter(cx<T>* v) {
  constexpr int R = 1 << LOGR, FIRST = LOGR % 2 ? 8 : 4;
  cx<T> x[R];
#pragma unroll
  for (int k = 0; k < R; ++k) x[k] = v[bitrev(k, LOGR)];
  if constexpr (LOGR % 2) {
#pragma unroll
    for (int k = 0; k < R; k += 2) {
      const cx<T> a = x[k], b = x[k + 1];
      x[k] = madd(a, unit128<T>(16), b);
      x[k + 1] = msub(a, unit128<T>(16), b);
    }
  }
#pragma unroll
  for (int len = FIRST; len <= R; len *= 4) {
    const int q = len / 4;
#pragma unroll
    for (int j = 0; j < q; ++j) {
      const int h = (4 * j + 1) * (32 / len);
#pragma unroll
      for (int k = j; k < R; k += len) {   // residues 0, 2, 1, 3 mod 4 of the sub-transforms, bit-reversed
        cx<T> a = x[k], c = x[k + q], b = x[k + 2 * q], d = x[k + 3 * q];
        bfly4(a, b, c, d, unit128<T>(h), unit128<T>(2 * h), unit128<T>(3 * h));
        x[k] = a;
        x[k + q] = b;
        x[k + 2 * q] = c;
        x[k + 3 * q] = d;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = x[k];
}

// Its transpose, X[n] = sum_k v[k] exp(-2 pi i n (k + 1/4) / R): the same levels in reverse
// order, a 4-point DFT followed by the twiddles
template <typename T, int LOGR>
__device__ __forceinline__ void dif_quarter(cx<T>* v) {
  constexpr int R = 1 << LOGR, FIRST = LOGR % 2 ? 8 : 4;
#pragma unroll
  for (int len = R; len >= FIRST; len /= 4) {
    const int q = len / 4;
#pragma unroll
    for (int j = 0; j < q; ++j) {
#pragma unroll
      for (int k = j; k < R; k += len) {
        const cx<T> a = v[k], b = v[k + q], c = v[k + 2 * q], d = v[k + 3 * q];
        const cx<T> t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = csub(b, d);
        const int h = (4 * j + 1) * (32 / len);
        v[k] = cadd(t0, t2);
        v[k + q] = cmul(csub(t0, t2), unit128<T>(2 * h));   // residue 2, in bit-reversed place
        v[k + 2 * q] = cmul(cx<T>{t1.re + t3.im, t1.im - t3.re}, unit128<T>(h));
        v[k + 3 * q] = cmul(cx<T>{t1.re - t3.im, t1.im + t3.re}, unit128<T>(3 * h));
      }
    }
  }
  if constexpr (LOGR % 2) {
#pragma unroll
    for (int k = 0; k < R; k += 2) {
      const cx<T> a = v[k], b = v[k + 1];
      v[k] = cadd(a, b);
      v[k + 1] = cmul(csub(a, b), unit128<T>(16));
    }
  }
  cx<T> x[R];
#pragma unroll
  for (int k = 0; k < R; ++k) x[k] = v[bitrev(k, LOGR)];
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = x[k];
}

// Plain 16-point DFT in registers, natural order in and out, as 4 x 4:
// X[k1 + 4 k2] = sum_n2 W_4^(n2 k2) [ W_16^(n2 k1) sum_n1 x[n2 + 4 n1] W_4^(n1 k1) ]
template <typename T>
__device__ __forceinline__ void dft4(cx<T>& a0, cx<T>& a1, cx<T>& a2, cx<T>& a3) {
  const cx<T> t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = csub(a1, a3);
  const cx<T> mt3 = {t3.im, -t3.re};   // -i t3
  a0 = cadd(t0, t2);
  a2 = csub(t0, t2);
  a1 = cadd(t1, mt3);
  a3 = csub(t1, mt3);
}

template <typename T>
__device__ __forceinline__ void dft16(cx<T>* v) {
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[n2 + 4], v[n2 + 8], v[n2 + 12]);   // v[n2 + 4 k1]
#pragma unroll
  for (int n2 = 1; n2 < 4; ++n2)
#pragma unroll
    for (int k1 = 1; k1 < 4; ++k1) v[n2 + 4 * k1] = twiddle_const(v[n2 + 4 * k1], n2 * k1, 16);
  cx<T> y[16];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    cx<T> a0 = v[4 * k1], a1 = v[4 * k1 + 1], a2 = v[4 * k1 + 2], a3 = v[4 * k1 + 3];
    dft4(a0, a1, a2, a3);
    y[k1] = a0;
    y[k1 + 4] = a1;
    y[k1 + 8] = a2;
    y[k1 + 12] = a3;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = y[k];
}

// 8-byte LDS slots: a float32 point, or one part of a float64 point
template <typename T> struct Slot;
template <> struct Slot<float> { using type = cx<float>; };
template <> struct Slot<double> { using type = double; };

// v[i] <- the value that wrote slot rd(i), where this lane's v[i] goes to slot wr(i); the
// slots belong to this wavefront
template <typename T, typename Wr, typename Rd>
__device__ __forceinline__ void exchange_private(cx<T>* v, typename Slot<T>::type* row, Wr wr, Rd rd) {
  if constexpr (sizeof(T) == 4) {
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) row[wr(i)] = v[i];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = row[rd(i)];
  } else {
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) row[wr(i)] = v[i].re;
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i].re = row[rd(i)];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) row[wr(i)] = v[i].im;
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i].im = row[rd(i)];
  }
}

// Workgroup exchange from columns to rows (TO_ROWS; v[c NO + k] of column g = t + NT c ->
// v[16 i + j] of row w + 16 i at l + 64 j) or back, in RPW halves of 16 rows.  Entered and
// left with the LDS rows free of readers other than their own wavefront.
template <typename T, int NO, int RPW, bool TO_ROWS>
__device__ __forceinline__ void exchange_rows(cx<T>* v, typename Slot<T>::type* lds, int t) {
  using S = WaveShape<NO, RPW>;
  if constexpr (S::NW == 1 && NO == 1) {
    return;   // a wavefront's columns l + 64 c are its row
  } else {
    constexpr int PARTS = sizeof(T) == 4 ? 1 : 2, H = S::NW;   // H rows in LDS at a time
    const int l = t & 63, w = t >> 6;
    // Two rows in registers: the rows beyond an LDS instruction's offset from a base of their own,
    // which the compiler does not see through (else it holds eight addresses instead of one over both
    // rows, beside 64 registers of points, and spills: 2^24 samples 71.1 us against 68.3 with this and
    // the rows' own addresses, 2^33 27.1 ms and 91.7 GB of traffic against 25.9 and 78.1)
    const int far = RPW == 2 ? (int)opaque((uint32_t)(t + 8 * kWRow)) : t;
    auto column = [&](int k, int c) {
      return RPW == 2 && k >= 8 ? far + (k - 8) * kWRow + S::NT * c : k * kWRow + t + S::NT * c;
    };
    cx<T> out[S::E];
#pragma unroll
    for (int i = 0; i < S::RPW; ++i)
#pragma unroll
      for (int part = 0; part < PARTS; ++part) {
        auto put = [&](int slot, cx<T> z) {
          if constexpr (sizeof(T) == 4) lds[slot] = z;
          else lds[slot] = part ? z.im : z.re;
        };
        auto get = [&](int slot, cx<T>& z) {
          if constexpr (sizeof(T) == 4) {
            z = lds[slot];
          } else {
            const T x = lds[slot];
            if (part) z.im = x; else z.re = x;
          }
        };
        if (i + part > 0) __syncthreads();   // the previous part's readers are done
        if constexpr (TO_ROWS) {
#pragma unroll
          for (int c = 0; c < S::C; ++c)
#pragma unroll
            for (int k = 0; k < H; ++k) put(column(k, c), v[c * NO + H * i + k]);
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) put(w * kWRow + l + 64 * j, v[16 * i + j]);
        }
        __syncthreads();
        if constexpr (TO_ROWS) {
#pragma unroll
          for (int j = 0; j < 16; ++j) get(w * kWRow + l + 64 * j, out[16 * i + j]);
        } else {
#pragma unroll
          for (int c = 0; c < S::C; ++c)
#pragma unroll
            for (int k = 0; k < H; ++k) get(column(k, c), out[c * NO + H * i + k]);
        }
      }
#pragma unroll
    for (int e = 0; e < S::E; ++e) v[e] = out[e];
  }
}

// Keeps the scheduler from hoisting later table loads over this point, where they would
// not fit in registers beside the transform and spill
__device__ __forceinline__ void sched_stop() { __builtin_amdgcn_sched_barrier(0); }

template <int n, typename T>
__device__ __forceinline__ void load_twiddles(cx<T>* w, const cx<T>* __restrict__ p) {
#pragma unroll
  for (int i = 0; i < n; ++i) w[i] = p[i];
}

template <typename T, int RPW>
constexpr bool wave_early = sizeof(T) == 4 && RPW == 1;
template <typename T, int NO, int RPW>
constexpr bool wave_itab = RPW == 2 || (sizeof(T) == 8 && NO >= 8);

// One row: 1024-point forward stage, symbol, 1024-point inverse stage and the twiddle
// before the inverse's outer stage.  v[j] = column l + 64 j of row k_o on entry and exit.
// EARLY: table loads go out a stage ahead, behind the exchange before it, and the symbol's
// before the stage that needs it; else (float64, or two rows in registers) where their values
// are used, and the last inverse stage's from itab, a copy in LDS ([8][64]), where workgroups are
// large enough for one (2^24 samples: float32 NO = 32 71.6 us against 83.1 from memory, float64 NO = 16 128
// against 131; for NO < 8 the copies would cost occupancy, 90 against 85 at NO = 1).
template <typename T, int NO, int RPW>
__device__ __forceinline__ void filter_row(cx<T>* v, typename Slot<T>::type* row, const cx<T>* __restrict__ tab,
                                           const T* __restrict__ sym, const cx<T>* itab, int k_o, int l) {
  using W = WaveTables<NO>;
  constexpr bool EARLY = wave_early<T, RPW>, TWO = RPW == 2;
  // Six operations in float64 and, with two rows in registers, in the third stage; in the inverse of
  // float32 but at NO = 1 and 2, where they would put the error above the plain transform's (1.05 of
  // it, 0.99 so, for 3 % more time), and there not in the 4-point stages of float64 either.  Eight
  // everywhere in float64 spill (NO = 1: 142 us against 82; an operator of 2 x 2^24 samples at
  // NO = 16, the 4-point stages alone: 599 against 517).
  constexpr bool SUM6 = sizeof(T) == 8, INV6 = sizeof(T) == 8 || NO > 2;
  if (TWO) l = (int)opaque((uint32_t)l);   // (each row forms its addresses anew)
  const int m = l & 15, hq = l >> 4;
  const cx<T>* __restrict__ t2 = tab + W::F2 + (uint32_t)((k_o * 16 + 4 * hq) * 2);
  const cx<T>* __restrict__ t3 = tab + W::F3 + (uint32_t)((k_o * 64 + l) * 8);
  const T* __restrict__ fs = sym + (uint32_t)(k_o * 1024 + l);
  cx<T> w2[8], w3[8];
  T f[16];
  if (EARLY) load_twiddles<8>(w2, t2);
  {   // forward: 16 points over j; the row's twiddles are uniform (scalar loads, all of them)
    const cx<T>* __restrict__ w1 = tab + W::F1 + k_o * 8;
    dit<T, 4, SUM6>(v, [&](int len, int j) { return w1[len == 2 ? 0 : len / 4 + j]; });
  }
  if (TWO) sched_stop();
  if (!EARLY) load_twiddles<8>(w2, t2);
  // (k1, l) -> lane (m, hq): k1 = 4 hq + e, h = 0 .. 3
  exchange_private<T>(v, row, [&](int i) { return i * 64 + l; },
                      [&](int i) { return (4 * hq + (i >> 2)) * 64 + m + 16 * (i & 3); });
  if (EARLY) load_twiddles<8>(w3, t3);
#pragma unroll
  for (int e = 0; e < 4; ++e) dit<T, 2, SUM6 && (NO > 2)>(v + 4 * e, [&](int len, int) { return w2[2 * e + len / 4]; });   // 4 points over h
  if (!EARLY) load_twiddles<8>(w3, t3);
  // (k1, c1, m) -> lane mu = k1 + 16 c1, register m
  exchange_private<T>(v, row, [&](int i) { return ((i & 3) * 16 + 4 * hq + (i >> 2)) * 17 + m; },
                      [&](int i) { return l * 17 + i; });
  if (EARLY) {
#pragma unroll
    for (int c = 0; c < 16; ++c) f[c] = fs[64 * c];
  }
  dit<T, 4, !EARLY>(v, [&](int len, int j) { return w3[len == 2 ? 0 : len / 4 + j]; });   // 16 points over m
#pragma unroll
  for (int c = 0; c < 16; ++c) {   // conj(F Z)
    if (!EARLY) f[c] = fs[64 * c];
    v[c] = {v[c].re * f[c], -(v[c].im * f[c])};
  }
  dft16<T>(v);   // inverse: 16 points over c2
  load_twiddles<2>(w2, tab + W::I2 + (uint32_t)(m * 2));
  // (c1, k1, m) -> lane (m, hq): k1 = 4 hq + e, c1 = 0 .. 3
  exchange_private<T>(v, row, [&](int i) { return l * 17 + i; },
                      [&](int i) { return ((i & 3) * 16 + 4 * hq + (i >> 2)) * 17 + m; });
  if (EARLY) load_twiddles<8>(w3, tab + W::I3 + (uint32_t)(l * 8));
#pragma unroll
  for (int e = 0; e < 4; ++e) dit<T, 2, INV6 && (NO > 2)>(v + 4 * e, [&](int len, int) { return w2[len / 4]; });   // 4 points over c1
  // (k1, l) -> lane l, register k1
  exchange_private<T>(v, row, [&](int i) { return (4 * hq + (i >> 2)) * 64 + m + 16 * (i & 3); },
                      [&](int i) { return i * 64 + l; });
  if constexpr (wave_itab<T, NO, RPW>) {
#pragma unroll
    for (int i = 0; i < 8; ++i) w3[i] = itab[i * 64 + l];
  } else if (!EARLY) {
    load_twiddles<8>(w3, tab + W::I3 + (uint32_t)(l * 8));
  }
  dit<T, 4, INV6>(v, [&](int len, int j) { return w3[len == 2 ? 0 : len / 4 + j]; });   // 16 points over k1
  const cx<T>* __restrict__ w4 = tab + W::I4 + (uint32_t)(k_o * 1024 + l);
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = cmul(v[j], w4[64 * j]);
}

// One workgroup per (chunk, RHS).  Workgroups are dealt to the 8 XCDs round-robin in linear
// (x-fastest) order, so XCD x takes workgroups x, x + 8, ...; it gets a contiguous run of
// (RHS, chunk) pairs instead, so that neighbouring chunks, whose windows overlap by 2 n_c
// samples, read the shared samples through the same L2.  16 wavefronts per CU (4 per SIMD)
// whatever NO: LDS holds 16 rows.
//
// SKY = 1 or 3: the window is looked up: yin is a map of SKY Stokes parameters (rows of stride
// sky.vs), sample t the value of pixel sky.idx[t] (-1: none) rounded to T, as the gather
// kernel would have stored it (the plan's sees_map says when, with both sides' times).
template <typename T, typename Tin, int NO, int RPW, int SKY>
__global__ __attribute__((amdgpu_flat_work_group_size(WaveShape<NO, RPW>::NT, WaveShape<NO, RPW>::NT),
                          amdgpu_waves_per_eu(4))) void k_ols_wave(
    const Tin* __restrict__ yin, T* __restrict__ yout, const OlsChunk* __restrict__ chunks,
    const T* __restrict__ spec, const cx<T>* __restrict__ tab, int64_t n_t, int n_c, int m,
    const CgState* __restrict__ st, SkyView sky) {
  using S = WaveShape<NO, RPW>;
  constexpr int N = S::N, NT = S::NT;
  constexpr int LOGNO = S::LOGNO;
  const int64_t n_wg = (int64_t)gridDim.x * gridDim.y;
  const int64_t wl = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t xq = n_wg >> 3, xr = n_wg & 7, xw = wl & 7;
  const int64_t job = xw * xq + (xw < xr ? xw : xr) + (wl >> 3);
  const int rhs = __builtin_amdgcn_readfirstlane((int)(job / gridDim.x));   // uniform: scalar row offsets
  if (st && !st[rhs].active) return;   // this RHS has stopped iterating
  __shared__ __align__(16) typename Slot<T>::type lds[S::LDS_SLOTS];
  __shared__ __align__(16) cx<T> itab[wave_itab<T, NO, RPW> ? 512 : 1];
  const OlsChunk ch = chunks[job - (int64_t)rhs * gridDim.x];
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  if constexpr (wave_itab<T, NO, RPW>)   // (the exchange before its first use has a barrier)
    for (int i = t; i < 512; i += NT) itab[(i & 7) * 64 + (i >> 3)] = tab[WaveTables<NO>::I3 + i];

  // the window: v[c NO + n_o] = x[n] - i x[n + N], n = t + NT c + 1024 n_o, x[i] = TOD sample
  // s0 + i inside the interval, else 0: window samples [a, b) are data, and a buffer over
  // them gives the zeros (every constant beside a column's offset is a multiple of 4096
  // bytes, which the instruction's offset field cannot hold)
  cx<T> v[S::E];
  T mean = (T)0;   // the window's offset (fft.hpp)
  const int64_t s0 = ch.out_start - n_c;
  const int a = (int)(ch.iv_lo > s0 ? ch.iv_lo - s0 : 0);   // (iv_lo <= out_start: a <= n_c)
  const int b = (int)(ch.iv_hi - s0 < 2 * N ? ch.iv_hi - s0 : 2 * N);
  if constexpr (SKY > 0) {
    const Rsrc ids = buffer_of(sky.idx + s0 + a, (b - a) * 4);
    const Rsrc ang = buffer_of(SKY == 3 ? sky.w + (s0 + a) : nullptr, SKY == 3 ? (b - a) * 8 : 0);
    const Tin* __restrict__ map = yin + (int64_t)rhs * sky.vs;
    if constexpr (S::NW > 1) mean = window_mean<T, 2 * N>(t, [&](int n) {
      const uint32_t k = (uint32_t)(n - a);
      int32_t p;
      float2 sc = make_float2(0.f, 0.f);
      buffer_get(ids, opaque(4 * k), p);
      if constexpr (SKY == 3) buffer_get(ang, opaque(8 * k), sc);
      p = k < (uint32_t)(b - a) ? p : -1;
      const double val = sky_value<SKY, Tin>(map, p >= 0 ? p : 0, sc.x, sc.y);
      return p >= 0 ? (T)val : (T)0;
    });
    constexpr int K = 2 * NO < 32 ? 2 * NO : 32;   // samples whose pixels are in registers at once
#pragma unroll
    for (int c = 0; c < S::C; ++c) {
      const uint32_t i = opaque((uint32_t)(t + NT * c - a));
#pragma unroll
      for (int e0 = 0; e0 < 2 * NO; e0 += K) {
        int32_t p[K];   // -1 outside the data (there the buffer reads 0)
#pragma unroll
        for (int e = 0; e < K; ++e) {
          const uint32_t k = i + 1024 * ((e0 + e) % NO) + ((e0 + e) / NO) * N;
          buffer_get(ids, 4 * k, p[e]);
          p[e] = k < (uint32_t)(b - a) ? p[e] : -1;
        }
#pragma unroll
        for (int e = 0; e < K; ++e) {
          const int n_o = (e0 + e) % NO, half = (e0 + e) / NO;
          float2 sc = make_float2(0.f, 0.f);
          if constexpr (SKY == 3) buffer_get(ang, 8 * (i + 1024 * n_o + half * N), sc);
          const double val = sky_value<SKY, Tin>(map, p[e] >= 0 ? p[e] : 0, sc.x, sc.y);
          const T x = p[e] >= 0 ? (T)val : (T)0;
          if (half) v[c * NO + n_o].im = -x; else v[c * NO + n_o].re = x;
        }
      }
    }
  } else {
    const Rsrc src = buffer_of(yin + (int64_t)rhs * n_t + s0 + a, (b - a) * (int)sizeof(Tin));
    if constexpr (S::NW > 1) mean = window_mean<T, 2 * N>(t, [&](int n) {
      Tin x;
      buffer_get(src, opaque((uint32_t)(n - a) * (uint32_t)sizeof(Tin)), x);
      return (T)x;
    });
#pragma unroll
    for (int c = 0; c < S::C; ++c) {
      const uint32_t off = opaque((uint32_t)(t + NT * c - a) * (uint32_t)sizeof(Tin));
#pragma unroll
      for (int n_o = 0; n_o < NO; ++n_o) {
        Tin x, y;
        buffer_get(src, off + 1024 * n_o * (uint32_t)sizeof(Tin), x);
        buffer_get(src, off + (1024 * n_o + N) * (uint32_t)sizeof(Tin), y);
        v[c * NO + n_o] = {(T)x, -(T)y};
      }
    }
  }
  if constexpr (S::NW == 1) {   // one wavefront: from eight runs of 64 samples
    T sum = (T)0, sq = (T)0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const cx<T> z = v[4 * i];
      sum += z.re - z.im;
      sq += z.re * z.re + z.im * z.im;
    }
    mean = offset_of<64>(sum, sq, 512);
  }
  if constexpr (RPW == 2) mean = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mean)));   // (the same in every lane)
#pragma unroll
  for (int e = 0; e < S::E; ++e) v[e] = {v[e].re - mean, v[e].im + mean};
  const T* __restrict__ sym = spec + (int64_t)ch.filter * (N + 1);
  // forward, outer stage over n_o
  if constexpr (NO > 1) {
#pragma unroll
    for (int c = 0; c < S::C; ++c) dit_quarter<T, LOGNO>(v + c * NO);
  }
  exchange_rows<T, NO, RPW, true>(v, lds, t);
  // the rows of this wavefront
#pragma unroll
  for (int i = 0; i < S::RPW; ++i)
    filter_row<T, NO, RPW>(v + 16 * i, lds + w * kWRow, tab, sym, itab, w + S::NW * i, t & 63);
  exchange_rows<T, NO, RPW, false>(v, lds, t);
  // inverse, outer stage over k_o; the outputs n and n + N of the window, positions
  // [n_c, n_c + m) of it from out_start on, cut at the interval's end
  const int len = (int)(ch.iv_hi - ch.out_start < m ? ch.iv_hi - ch.out_start : m);
  const Rsrc dst = buffer_of(yout + (int64_t)rhs * n_t + ch.out_start, len * (int)sizeof(T));
  const T back = mean * sym[N];   // what the filter makes of the mean
#pragma unroll
  for (int c = 0; c < S::C; ++c) {
    if constexpr (NO > 1) dif_quarter<T, LOGNO>(v + c * NO);
    const uint32_t off = opaque((uint32_t)(t + NT * c - n_c) * (uint32_t)sizeof(T));
#pragma unroll
    for (int n_b = 0; n_b < NO; ++n_b) {
      const cx<T> z = v[c * NO + n_b];
      buffer_put(dst, off + 1024 * n_b * (uint32_t)sizeof(T), z.re + back);
      buffer_put(dst, off + (1024 * n_b + N) * (uint32_t)sizeof(T), z.im + back);
    }
  }
}

// Twiddle tables from float64 angles
template <typename T, int NO>
__global__ void k_wave_tables(cx<T>* __restrict__ tab) {
  using W = WaveTables<NO>;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= W::TOTAL) return;
  // entry i of a stage with shift num / den, as a fraction of a turn: num / (den 2^(i + 1))
  auto stage = [](int i, double num, double den) -> double { return num / (den * (double)(2 << i)); };
  // entry i of a 16-point stage
  auto stage16 = [](int i, double num, double den) -> double {
    const int len = i == 0 ? 2 : i == 1 ? 4 : i < 4 ? 8 : 16, j = i == 0 ? 0 : i - len / 4;
    return (j * den + num) / ((double)len * den);
  };
  double frac;
  if (e < W::F2) {
    frac = stage16(e % 8, e / 8 + 0.25, NO);
  } else if (e < W::F3) {
    const int i = e - W::F2, k_o = i / 32, k1 = (i / 2) % 16;
    frac = stage(i % 2, k_o + 0.25 + (double)NO * k1, 16.0 * NO);
  } else if (e < W::I2) {
    const int i = e - W::F3, k_o = i / 512, mu = (i / 8) % 64;
    frac = stage16(i % 8, k_o + 0.25 + (double)NO * mu, 64.0 * NO);
  } else if (e < W::I3) {
    const int i = e - W::I2;
    frac = stage(i % 2, i / 2, 16.0);
  } else if (e < W::I4) {
    const int i = e - W::I3;
    frac = stage16(i % 8, i / 8, 64.0);
  } else {
    const int i = e - W::I4, k_o = i / 1024, g = i % 1024;
    frac = (double)(g * (4 * k_o + 1)) / (4096.0 * NO);
  }
  double sn, cs;
  sincospi(2.0 * frac, &sn, &cs);
  tab[e] = {(T)cs, (T)(-sn)};
}

template <typename T, int NO>
hipError_t tables_launch(void* tab, hipStream_t s) {
  constexpr int n = WaveTables<NO>::TOTAL;
  hipLaunchKernelGGL((k_wave_tables<T, NO>), dim3((n + 255) / 256), dim3(256), 0, s, (cx<T>*)tab);
  return hipGetLastError();
}

template <typename T, typename Tin, int NO, int SKY = 0>
hipError_t wave_launch(const void* y_in, void* y_out, const OlsChunk* chunks, int n_chunks, const void* spec,
                       const void* tab, int64_t n_t, int n_c, int m, int n_rhs, hipStream_t s, const CgState* st,
                       const SkyView& sky = {}) {
  constexpr int RPW = NO == 32 ? 2 : 1;   // (16 wavefronts at most)
  hipLaunchKernelGGL((k_ols_wave<T, Tin, NO, RPW, SKY>), dim3((unsigned)n_chunks, (unsigned)n_rhs),
                     dim3(WaveShape<NO, RPW>::NT), 0, s, (const Tin*)y_in, (T*)y_out, chunks, (const T*)spec,
                     (const cx<T>*)tab, n_t, n_c, m, st, sky);
  return hipGetLastError();
}

// NO = 2^(logn - 10) of the lengths that exist: 2^10 .. 2^15 points in float32, .. 2^14 in float64
template <typename T, typename F>
auto wave_dispatch(int logn, F&& f) {
  switch (logn) {
    case 10: return f(std::integral_constant<int, 1>{});
    case 11: return f(std::integral_constant<int, 2>{});
    case 12: return f(std::integral_constant<int, 4>{});
    case 13: return f(std::integral_constant<int, 8>{});
    case 14: return f(std::integral_constant<int, 16>{});
    default:
      if constexpr (sizeof(T) == 4) return f(std::integral_constant<int, 32>{});
      else return f(std::integral_constant<int, 16>{});
  }
}

}  // namespace

bool ols_wave_exists(int logn, bool fp64) { return logn >= 10 && logn <= (fp64 ? 14 : 15); }

int ols_wave_table_count(int logn) {
  return wave_dispatch<float>(logn, [](auto no) -> int { return WaveTables<decltype(no)::value>::TOTAL; });
}

hipError_t launch_wave_tables(int logn, bool fp64, void* tab, hipStream_t s) {
  if (!ols_wave_exists(logn, fp64)) return hipErrorInvalidValue;
  if (fp64)
    return wave_dispatch<double>(logn, [&](auto no) -> hipError_t { return tables_launch<double, decltype(no)::value>(tab, s); });
  return wave_dispatch<float>(logn, [&](auto no) -> hipError_t { return tables_launch<float, decltype(no)::value>(tab, s); });
}

hipError_t launch_ols_wave(int logn, bool fp64, bool in_f64, const void* y_in, void* y_out, const OlsChunk* chunks,
                           int n_chunks, const void* spec, const void* tab, int64_t n_t, int n_c, int m, int n_rhs,
                           hipStream_t s, const CgState* st) {
  if (!ols_wave_exists(logn, fp64)) return hipErrorInvalidValue;
  if (n_chunks == 0 || n_rhs == 0) return hipSuccess;
  auto go = [&](auto tc, auto tin) -> hipError_t {
    using T = decltype(tc);
    using Tin = decltype(tin);
    return wave_dispatch<T>(logn, [&](auto no) -> hipError_t {
      return wave_launch<T, Tin, decltype(no)::value>(y_in, y_out, chunks, n_chunks, spec, tab, n_t, n_c, m, n_rhs, s,
                                                      st);
    });
  };
  if (fp64) return in_f64 ? go(double{}, double{}) : go(double{}, float{});
  return in_f64 ? go(float{}, double{}) : go(float{}, float{});
}

hipError_t launch_ols_sky(int logn, bool fp64, bool map_f64, int ns, const void* map, const SkyView& sky, void* y_out,
                          const OlsChunk* chunks, int n_chunks, const void* spec, const void* tab, int64_t n_t, int n_c,
                          int m, int n_rhs, hipStream_t s, const CgState* st) {
  if (!ols_wave_exists(logn, fp64)) return hipErrorInvalidValue;
  if (n_chunks == 0 || n_rhs == 0) return hipSuccess;
  auto go = [&](auto tc, auto tin) -> hipError_t {
    using T = decltype(tc);
    using Tin = decltype(tin);
    return wave_dispatch<T>(logn, [&](auto no) -> hipError_t {
      constexpr int NO = decltype(no)::value;
      return ns == 1 ? wave_launch<T, Tin, NO, 1>(map, y_out, chunks, n_chunks, spec, tab, n_t, n_c, m, n_rhs, s, st, sky)
                     : wave_launch<T, Tin, NO, 3>(map, y_out, chunks, n_chunks, spec, tab, n_t, n_c, m, n_rhs, s, st, sky);
    });
  };
  if (fp64) return map_f64 ? go(double{}, double{}) : hipErrorInvalidValue;
  return map_f64 ? go(float{}, double{}) : go(float{}, float{});
}

}  // namespace mm
