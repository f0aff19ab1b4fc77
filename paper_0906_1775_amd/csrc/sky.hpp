// One sample of a map seen through the pointing (the sky gather, and the small maps' filter,
// which reads its windows this way).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace mm {

// The (I, Q, U) values of one pixel, read as one load
template <typename Tp> struct Stokes3 { Tp v[3]; };

// y_t = sum_s w_ts p_{pix_t, s} for the samples of row r; o must be a valid pixel:
// excised samples are clamped to pixel 0 by the caller and their value discarded,
// so that no lookup waits behind a branch.
template <int NS, typename Tp>
__device__ __forceinline__ double sky_value(const Tp* __restrict__ row, int32_t o, float s, float c) {
  if constexpr (NS == 1) {
    return (double)row[o];
  } else {
    const Stokes3<Tp> m = *reinterpret_cast<const Stokes3<Tp>*>(row + (int64_t)o * 3);
    return 0.5 * ((double)m.v[0] + (double)s * (double)m.v[1] + (double)c * (double)m.v[2]);
  }
}

}  // namespace mm
