// Order of the observed pixels.  Maps are usually rasters, and pixels that are neighbours on the
// sky along either axis are hit by neighbouring samples of some detector.  Where the TOD shows
// the row length of the raster, the pixels are kept by 8 x 8 tiles (tiles row by row, inside a
// tile by the interleaved bits of both coordinates), so that the 64 pixels of a scatter slice
// and the samples a gather wavefront looks up share cache lines along both axes.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace mm {

struct Raster {
  uint32_t w = 0;    // row length; 0 = no raster known, pixels in their own order
  uint32_t wt = 0;   // tiles per row
};

__host__ __device__ inline uint32_t spread3(uint32_t v) { return (v & 1) | (v & 2) << 1 | (v & 4) << 2; }
__host__ __device__ inline uint32_t gather3(uint32_t v) { return (v & 1) | (v >> 1 & 2) | (v >> 2 & 4); }

// sort key of pixel p, and the pixel of a key
__host__ __device__ inline uint32_t raster_key(Raster r, uint32_t p) {
  if (r.w == 0) return p;
  const uint32_t y = p / r.w, x = p - y * r.w;
  return ((y >> 3) * r.wt + (x >> 3)) << 6 | spread3(x) | spread3(y) << 1;
}
__host__ __device__ inline uint32_t raster_pixel(Raster r, uint32_t k) {
  if (r.w == 0) return k;
  const uint32_t tile = k >> 6, ty = tile / r.wt, tx = tile - ty * r.wt;
  return (ty * 8 + gather3(k >> 1)) * r.w + tx * 8 + gather3(k);
}

}  // namespace mm
