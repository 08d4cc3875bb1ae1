// conv_smallc4.hip -- first-layer forward for four input channels (gfx950).
//
// The scaled-up network's first layer (3^3 taps, 4 -> 16 channels, stride 1)
// contracts K = 27 taps x 4 channels.  The four channels of a voxel are 8
// bytes in bf16 and 16 bytes in fp32, so an MFMA operand fragment is made of
// whole voxels and no element is ever moved by itself:
//   bf16  v_mfma_f32_16x16x32: lane (row r, K quarter g) needs eight K values
//         = two taps; MFMA m holds taps 8 m .. 8 m + 7, lane quarter g taps
//         8 m + 2 g and the next.  The fused form carries the bias in two spare
//         slots of the last MFMA (tap 27) against ones, as bf16(b) and the
//         bf16 rounding of the rest.  These are the K order and the roundings
//         of the general first-layer kernel: the outputs are bit for bit its own.
//   fp32  v_mfma_f32_16x16x4: the four K slots of MFMA t are the channels of
//         tap t, the order of the generic kernel (the same sums bit for bit);
//         every tap is one 4-byte read at a compile-time offset.
// bf16 slots past the last tap read zeros (an LDS area that no tile writes; the
// lanes that hold them leave out the row's offset), so an infinity or NaN of the
// input reaches exactly the outputs whose window holds it, and as itself.
//
// Voxel order inside a tile: row r = 4 q + j is (h = j >> 1, w = 2 q + (j & 1))
// and two tiles (dd = 0, 1) make the 2 x 2 x 8 voxels of four pooling windows;
// the accumulator layout then leaves each window in one lane.  The slope ballots
// go to two registers (even and odd voxels) by lane writes, 16 lanes to each of
// the four (dd, hh) rows, and two byte permutes put them into the mask tensor's
// order.
//
// Persistent workgroups (four per compute unit: 39.8 KB of LDS in bf16, 37.5 in
// fp32, and at most 128 registers each) form the weight fragments once; tiles go
// to the XCDs in contiguous runs.
// Bound by vector issue (45 instructions per 32 voxels, and about 20 more for
// staging) beside the MFMAs in bf16, by the matrix core in fp32.  256^3 batch 2
// bf16: 926 us with the general kernel's element gathers, 211-233 us here
// (470 MB of tensor traffic: 94 us at a copy's rate); fp32 100^3 batch 4: 192 us
// against about 540 us of the generic kernel.

#include "cf_common.h"
#include "cf_kernels.h"
#include "conv_smallc4_halo.h"

#include <algorithm>

// v_writelane_b32 through the compiler (it places the wait states between the
// compare that writes a ballot and the move that reads it)
__device__ int cf_lane_write4(int v, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace cf {
namespace {

template <int DT> struct C4Geom {
  static constexpr int VB = DT == DT_BF16 ? 8 : 16;     // bytes of a voxel
  static constexpr int TW = DT == DT_BF16 ? 64 : 32;    // output tile along w
  // row pitch: the two h rows of a read sit in disjoint banks
  static constexpr int RP = DT == DT_BF16 ? 576 : 640;
};

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2a2_t __attribute__((ext_vector_type(2), aligned(2)));

template <int DT, bool FUSED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void l1c4_fwd_kernel(
    const typename Store<DT>::T *__restrict__ x, const typename Store<DT>::T *__restrict__ w,
    const float *__restrict__ bias, float alpha, typename Store<DT>::T *__restrict__ out,
    uint16_t *__restrict__ mask16, SmallcParams p, C4Tiles tiles, int total_tiles) {
  using G = C4Geom<DT>;
  constexpr bool BF = DT == DT_BF16;
  constexpr int TW = G::TW, RP = G::RP, VB = G::VB;
  // bf16: zeros behind the halo, as far as a row's reads reach from their address
  constexpr int HB = C4HD * C4HH * RP, ZB = BF ? (C4HH * RP + (TW - 8) * VB + VB + 15) / 16 * 16 : 0;
  __shared__ __attribute__((aligned(16))) unsigned char halo[HB + ZB];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;

#pragma unroll
  for (int k = 0; k < ZB; k += 256 * 16)
    if (k + 16 * tid < ZB) *reinterpret_cast<u32x4_t *>(halo + HB + k + 16 * tid) = u32x4_t{0u, 0u, 0u, 0u};

  // ---- tap slots of this lane: LDS offsets (from the tile row's first voxel) and weights
  const int voff = (((r & 3) >> 1) * RP) + (2 * (r >> 2) + (r & 1)) * VB;
  int a0[4], a1[4];
  bf16x8_t bwb[4];
  float bwf[BF ? 1 : 27];
  auto tap_off = [](int t) { return ((t / 9) * C4HH + (t / 3) % 3) * RP + (t % 3) * VB; };
  if constexpr (BF) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int s = 4 * m + g;
      const int t0 = 2 * s, t1 = 2 * s + 1;
      const bool ok0 = t0 < 27, ok1 = t1 < 27;
      a0[m] = ok0 ? voff + tap_off(t0) : HB;
      a1[m] = ok1 ? voff + tap_off(t1) : HB;
      Vec16<DT_BF16> v;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        v.e[c] = ok0 ? w[(4 * t0 + c) * 16 + r] : (uint16_t)0;
        v.e[4 + c] = ok1 ? w[(4 * t1 + c) * 16 + r] : (uint16_t)0;
      }
      if (FUSED && s == 13) {  // tap 27: the bias
        const float b = bias[r];
        v.e[4] = f2bf(b);
        v.e[5] = f2bf(b - bf2f(v.e[4]));
      }
      bwb[m] = __builtin_bit_cast(bf16x8_t, v.u);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 27; ++t) bwf[t] = (float)w[(4 * t + g) * 16 + r];
  }

  C4Halo<TW, VB> hl;
  hl.init(tid, p);
  // tiles in eight contiguous runs, one per XCD (workgroup b runs on XCD b % 8)
  const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, nwg = gridDim.x >> 3;
  const int per = (total_tiles + 7) >> 3;
  const int tend = min(total_tiles, (xcd + 1) * per);
  for (int tile = xcd * per + wg; tile < tend; tile += nwg) {
    const C4Tile tl = c4_tile(tile, tiles, TW);
    const int n = tl.n, od0 = tl.d, oh0 = tl.h, ow0 = tl.w;
    u32x4_t hv[C4Halo<TW, VB>::NL];
    hl.load(x, p, tl, hv);
    __syncthreads();  // every wave has left the last tile
#pragma unroll
    for (int k = 0; k < C4Halo<TW, VB>::NL; ++k)
      if (tid + 256 * k < C4Halo<TW, VB>::ITEMS)
        *reinterpret_cast<u32x4_t *>(halo + (hl.pk[k] & 63) * RP + (hl.pk[k] >> 8) * 16) = hv[k];
    __syncthreads();

    for (int ri = wave; ri < (C4TD / 2) * (C4TH / 2); ri += 4) {
      const int bd = ri / (C4TH / 2), bh = ri % (C4TH / 2);
      const int vd0 = od0 + 2 * bd, vh0 = oh0 + 2 * bh;
      if (vd0 >= p.od || vh0 >= p.oh) continue;
      const int rb = (2 * bd * C4HH + 2 * bh) * RP;  // the brick row's first halo row
      int b0[4], b1[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        b0[m] = BF ? a0[m] + (m < 3 || g < 2 ? rb : 0) : 0;
        b1[m] = BF ? a1[m] + (m < 3 || g < 1 ? rb : 0) : 0;
      }
      uint32_t me = 0, mo = 0;  // lane 16 (2 dd + hh) + 2 seg + half: ballots of even / odd voxels
      const int pd_ = vd0 >> 1, ph_ = vh0 >> 1;
      const bool prow_ok = pd_ < p.pod && ph_ < p.poh;
      typename Store<DT>::T *const prow =
          out + ((((long long)n * p.pod + pd_) * p.poh + ph_) * p.pow_ + (ow0 >> 1) + g) * 16 + r;
#pragma unroll
      for (int sg = 0; sg < TW / 8; ++sg) {
        if (ow0 + 8 * sg >= p.ow) break;
        f32x4_t acc[2];
#pragma unroll
        for (int dd = 0; dd < 2; ++dd) {
          acc[dd] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          const unsigned char *hs = halo + dd * C4HH * RP + 8 * sg * VB;
          if constexpr (BF) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const u32x2_t lo = *reinterpret_cast<const u32x2_t *>(hs + b0[m]);
              const u32x2_t hi = *reinterpret_cast<const u32x2_t *>(hs + b1[m]);
              u32x4_t av = {lo[0], lo[1], hi[0], hi[1]};
              if (FUSED && m == 3) av[2] = g == 1 ? 0x3f803f80u : av[2];  // the bias slots' ones
              acc[dd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av), bwb[m], acc[dd], 0, 0, 0);
            }
          } else {
#pragma unroll
            for (int t = 0; t < 27; ++t)
              acc[dd] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  *reinterpret_cast<const float *>(hs + rb + voff + 4 * g + tap_off(t)), bwf[t], acc[dd], 0, 0, 0);
          }
        }
        // this lane: channel r, rows 4 g + j -> voxel (hh = j >> 1, w = 8 sg + 2 g + (j & 1))
        if constexpr (FUSED) {
          float s = 0.f;
#pragma unroll
          for (int dd = 0; dd < 2; ++dd)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float u = acc[dd][j];
              const bool pos = u > 0.f;
              const uint64_t bal = __builtin_amdgcn_ballot_w64(pos);
              const int l0 = 16 * (2 * dd + (j >> 1)) + 2 * sg;
              uint32_t &mw = (j & 1) ? mo : me;
              mw = cf_lane_write4((int)(uint32_t)bal, l0, (int)mw);
              mw = cf_lane_write4((int)(uint32_t)(bal >> 32), l0 + 1, (int)mw);
              s = fmaf(pos ? 1.f : alpha, u, s);
            }
          if (prow_ok && (ow0 >> 1) + 4 * sg + g < p.pow_) prow[4 * sg * 16] = from_f32<DT>(s * 0.125f);
        } else {
#pragma unroll
          for (int dd = 0; dd < 2; ++dd)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int vd = vd0 + dd, vh = vh0 + (j >> 1), vw = ow0 + 8 * sg + 2 * g + (j & 1);
              if (vd < p.od && vh < p.oh && vw < p.ow)
                out[((((long long)n * p.od + vd) * p.oh + vh) * p.ow + vw) * 16 + r] = from_f32<DT>(acc[dd][j]);
            }
        }
      }
      if constexpr (FUSED) {
        // lane: voxels ow0 + 4 (lane % 16) .. + 3 of row (dd, hh) = lane / 16
        const int vd = vd0 + (lane >> 5), vh = vh0 + ((lane >> 4) & 1), vw = ow0 + 4 * (lane & 15);
        if (vd < p.od && vh < p.oh && vw < p.ow && 4 * (lane & 15) < TW) {
          const u32x2_t mv = {__builtin_amdgcn_perm(mo, me, 0x05040100u), __builtin_amdgcn_perm(mo, me, 0x07060302u)};
          uint16_t *mrow = mask16 + (((long long)n * p.od + vd) * p.oh + vh) * p.ow + vw;
          if (vw + 4 <= p.ow) {
            *reinterpret_cast<u32x2a2_t *>(mrow) = mv;  // 2-byte aligned where the row length is odd
          } else {
            mrow[0] = (uint16_t)mv[0];
            if (vw + 1 < p.ow) mrow[1] = (uint16_t)(mv[0] >> 16);
            if (vw + 2 < p.ow) mrow[2] = (uint16_t)mv[1];
          }
        }
      }
    }
  }
}

template <int DT, bool FUSED>
hipError_t launch_c4(const ConvShape &s, const void *x, const void *w, const float *bias, float alpha, void *out,
                     uint16_t *mask, hipStream_t st) {
  using T = typename Store<DT>::T;
  long long total;
  const C4Tiles tiles = c4_tiles(s, C4Geom<DT>::TW, &total);
  // four workgroups per compute unit stay resident; a multiple of the eight XCDs
  const int blocks = (int)std::min<long long>((total + 7) / 8 * 8, 4 * kNumCUs);
  hipLaunchKernelGGL((l1c4_fwd_kernel<DT, FUSED>), dim3(blocks), dim3(256), 0, st, (const T *)x, (const T *)w, bias,
                     alpha, (T *)out, mask, c4_params(s), tiles, (int)total);
  return hipGetLastError();
}

}  // namespace

// four input channels, 3^3, 16 outputs, stride 1; a tile count and halo offsets below
// 2^31 (inputs of more than 44 M voxels in an h w slice stay with the general kernels)
bool l1c4_supported(const ConvShape &s) {
  long long total;
  c4_tiles(s, 32, &total);
  if (total >= 0x7ffffff0LL || !c4_halo_fits(s)) return false;
  return s.ci == 4 && s.co == 16 && s.kd == 3 && s.kh == 3 && s.kw == 3 && s.sd == 1 && s.sh == 1 && s.sw == 1 &&
         s.pd <= 2 && s.ph <= 2 && s.pw <= 2;
}

hipError_t launch_conv_fwd_l1c4(const ConvShape &s, const void *x, const void *w, const float *bias, float alpha,
                                void *out, uint16_t *mask, bool fused, hipStream_t st) {
  if (s.dtype == DT_BF16)
    return fused ? launch_c4<DT_BF16, true>(s, x, w, bias, alpha, out, mask, st)
                 : launch_c4<DT_BF16, false>(s, x, w, bias, alpha, out, mask, st);
  if (fused) return hipErrorInvalidValue;
  return launch_c4<DT_F32, false>(s, x, w, bias, alpha, out, mask, st);
}

}  // namespace cf
