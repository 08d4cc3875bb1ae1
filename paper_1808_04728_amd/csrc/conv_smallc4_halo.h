// conv_smallc4_halo.h -- input halo of a 4 x 8 x TW output tile of the
// four-channel first layer, loaded into registers (gfx950).
//
// The 6 x 10 halo rows of TW + 2 voxels (VB bytes each) are cut into 16-byte
// chunks, dealt to the 256 threads once; a chunk's byte offset from the halo's
// first voxel never changes, so a persistent kernel keeps it in a register.
// Per tile one scalar bit mask says which rows lie outside the input, and a
// chunk whose row or column does is sent past the buffer's range by bit 31 of
// its offset: the load returns the zero padding.  Tiles that touch the left or
// right edge load the chunk's two voxels (bf16) one by one.
#pragma once

#include "cf_common.h"
#include "cf_kernels.h"
#include "fastdiv.h"

namespace cf {

constexpr int C4TD = 4, C4TH = 8;                // output tile (d, h)
constexpr int C4HD = C4TD + 2, C4HH = C4TH + 2;  // halo rows
constexpr int C4ROWS = C4HD * C4HH;
static_assert(C4ROWS <= 63, "one mask bit per halo row, bit 63 for idle chunks");

struct C4Tile {  // a tile's sample and first output voxel
  int n, d, h, w;
};

// tile order: w fastest, then h, d, sample
struct C4Tiles {
  FastDiv fw, fh, fd;
};

__device__ __forceinline__ C4Tile c4_tile(int tile, const C4Tiles &T, int tw) {
  const int a = fdiv(tile, T.fw), b = fdiv(a, T.fh), c = fdiv(b, T.fd);
  return C4Tile{c, (b - c * (int)T.fd.div) * C4TD, (a - b * (int)T.fh.div) * C4TH, (tile - a * (int)T.fw.div) * tw};
}

template <int TW, int VB> struct C4Halo {
  static constexpr int NV = TW + 2, NC = NV * VB / 16;
  static constexpr int ITEMS = C4ROWS * NC, NL = (ITEMS + 255) / 256;
  static_assert(NV * VB % 16 == 0, "whole chunks");
  uint32_t off[NL];  // byte offset of this thread's chunks from the halo's first voxel
  int pk[NL];        // halo row | chunk << 8 (row 63: idle)

  __device__ __forceinline__ void init(int tid, const SmallcParams &p) {
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int e = tid + 256 * k;
      const int v = e % NC, rb = e / NC;
      off[k] = (uint32_t)((((rb / C4HH) * p.h + rb % C4HH) * p.w) * VB + 16 * v);
      pk[k] = (e < ITEMS ? rb : 63) | v << 8;
    }
  }

  __device__ __forceinline__ void load(const void *x, const SmallcParams &p, const C4Tile &t, u32x4_t (&hv)[NL]) const {
    const int d0 = t.d - p.pd, h0 = t.h - p.ph, w0 = t.w - p.pw;
    // bit 10 a + b set: halo row (a, b) lies outside the input
    const int blo = h0 < 0 ? -h0 : 0, bhi = min(C4HH, p.h - h0);
    const uint64_t okh = ((1ull << bhi) - 1) & ~((1ull << blo) - 1);
    uint64_t ok = 0;
#pragma unroll
    for (int a = 0; a < C4HD; ++a)
      if ((unsigned)(d0 + a) < (unsigned)p.d) ok |= okh << (C4HH * a);
    const uint64_t bad = ~ok;
    // (the base may lie before the tensor; chunks there are masked)
    const char *base = (const char *)x + ((((long long)t.n * p.d + d0) * p.h + h0) * p.w + w0) * VB;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, 0x7fffffff, 0x00020000);
    if (w0 >= 0 && w0 + NV <= p.w) {
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const uint32_t o = off[k] | (uint32_t)(bad >> (pk[k] & 63)) << 31;
        hv[k] = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
      }
    } else {
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const uint32_t o = off[k] | (uint32_t)(bad >> (pk[k] & 63)) << 31;
        if constexpr (VB == 8) {
          typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
          const int c0 = w0 + 2 * (pk[k] >> 8);
          const u32x2_t lo = __builtin_amdgcn_raw_buffer_load_b64(
              r, o | (uint32_t)((unsigned)c0 >= (unsigned)p.w) << 31, 0, 0);
          const u32x2_t hi = __builtin_amdgcn_raw_buffer_load_b64(
              r, (o + 8) | (uint32_t)((unsigned)(c0 + 1) >= (unsigned)p.w) << 31, 0, 0);
          hv[k] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
        } else {
          const int c0 = w0 + (pk[k] >> 8);
          hv[k] = __builtin_amdgcn_raw_buffer_load_b128(r, o | (uint32_t)((unsigned)c0 >= (unsigned)p.w) << 31, 0, 0);
        }
      }
    }
  }
};

// what the offsets above need: every chunk of a tile's halo within 2^31 bytes of its first voxel
inline bool c4_halo_fits(const ConvShape &s) {
  const long long vb = s.dtype == DT_BF16 ? 8 : 16;
  return ((long long)C4HD * s.h + C4HH) * s.w * vb < (1LL << 31);
}

inline C4Tiles c4_tiles(const ConvShape &s, int tw, long long *total) {
  const int nw = (s.ow + tw - 1) / tw, nh = (s.oh + C4TH - 1) / C4TH, nd = (s.od + C4TD - 1) / C4TD;
  *total = (long long)s.n * nw * nh * nd;
  return C4Tiles{make_fastdiv(nw), make_fastdiv(nh), make_fastdiv(nd)};
}

inline SmallcParams c4_params(const ConvShape &s) {
  SmallcParams p{};
  p.n = s.n; p.d = s.d; p.h = s.h; p.w = s.w; p.ci = s.ci; p.co = s.co;
  p.kd = s.kd; p.kh = s.kh; p.kw = s.kw; p.pd = s.pd; p.ph = s.ph; p.pw = s.pw;
  p.od = s.od; p.oh = s.oh; p.ow = s.ow;
  p.pod = s.od / 2; p.poh = s.oh / 2; p.pow_ = s.ow / 2;
  return p;
}

}  // namespace cf
