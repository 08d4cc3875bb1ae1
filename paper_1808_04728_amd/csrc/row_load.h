// row_load.h -- eight consecutive 16-bit elements of a row that need not start
// on any alignment, zero outside the row (gfx950): bf16 voxels of a one-channel
// input, 16-channel slope mask words.
#pragma once

#include "cf_common.h"

namespace cf {

typedef uint32_t u32x4a2_t __attribute__((ext_vector_type(4), aligned(2)));

// voxels c0 .. c0 + 7 of the row xr of w >= 8 voxels.  A run that hangs over
// an end is read where it fits and moved into place (the row's neighbours in
// memory are never read), so a row of any length costs one load.
__device__ __forceinline__ u32x4_t load_run8(const uint16_t *xr, int c0, int w) {
  const int c = min(max(c0, 0), w - 8);
  const int dl = c0 - c;  // 0 inside; > 0 past the right end, < 0 before the left
  if (dl >= 8 || dl <= -8) return u32x4_t{0u, 0u, 0u, 0u};
  const u32x4_t v = *reinterpret_cast<const u32x4a2_t *>(xr + c);
  if (dl == 0) return v;
  uint64_t lo = v[0] | (uint64_t)v[1] << 32, hi = v[2] | (uint64_t)v[3] << 32;
  if (dl > 0) {  // element j <- j + dl
    const int s = 16 * dl;
    lo = s < 64 ? (lo >> s) | (hi << (64 - s)) : hi >> (s - 64);
    hi = s < 64 ? hi >> s : 0;
  } else {
    const int s = -16 * dl;
    hi = s < 64 ? (hi << s) | (lo >> (64 - s)) : lo << (s - 64);
    lo = s < 64 ? lo << s : 0;
  }
  return u32x4_t{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// the mask words of voxels c0 .. c0 + 7 (from m on) of a row of w > c0 voxels.  Past
// its end only the row's own words are read (the last row ends at the end of the
// buffer); those voxels pool into no window, so their bits may be anything.
__device__ __forceinline__ u32x4_t load_mask8(const uint16_t *m, int c0, int w) {
  if (c0 + 8 <= w) return *reinterpret_cast<const u32x4a2_t *>(m);
  uint32_t h[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) h[u] = c0 + u < w ? m[u] : 0u;
  return u32x4_t{h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16};
}

}  // namespace cf
