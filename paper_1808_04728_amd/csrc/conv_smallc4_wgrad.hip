// conv_smallc4_wgrad.hip -- backward weights of the four-channel first layer
// (3^3 taps, 4 -> 16 channels, stride 1, bf16, pooled), gfx950.
//
//   dW[(t, ci), co] = sum_v x~[v + t, ci] dz[v, co],  db[co] = sum_v dz[v, co]
// with dz rebuilt from the pooled-output gradient g and the slope mask,
//   dz = g[pool(v)] / 8 * (bit ? 1 : alpha)   (0 outside the pooling windows).
//
// The contraction runs over voxels (K), so both operands need eight
// consecutive voxels of one row per lane.
//   A: the input halo lies in LDS as it does in memory, 8 bytes (four channels)
//      a voxel.  In the transposing read (ds_read_b64_tr_b16) a lane's 8-byte
//      piece is one voxel, so pieces are tap columns kw and the result lane
//      4 kw + ci holds four consecutive voxels of channel ci: two reads make
//      the fragment of one (kd, kh) kernel row (12 of 16 rows used) with no
//      shifted copies.  A halo row serves every (voxel row, kernel row) pair
//      that meets there: the four voxel rows of a pooling window take 16
//      fragments for 36 products.
//   B: pooled values of one channel come from the same transposing read, once
//      as g and once as the rounded alpha g; doubled along w, the mask bit
//      picks one of them per voxel (one bit select per pair).  This is the
//      bf16 rounding of dz times 8.
// db is summed from the unrounded values: a fragment of ones times g and times
// the masked g, combined as alpha / 8 and (1 - alpha) / 8.  For a slope above 1
// that is a difference of large terms (and of infinities), for a slope of 0 an
// infinity of g meets the factor 0: there the workgroups whose sums call for it
// add up their dz once more, voxel by voxel (DEF, an instantiation of its own:
// its registers cost 1 to 2% of the launch, 128^3 batch 2 38.3 -> 39.1 us, and
// the pass itself 22% at a slope of 3).
//
// 256^3 batch 2: 1374 us with the general kernel (shifted copies built element
// by element, 79 KB of LDS), 235-252 us here.  Four workgroups per compute unit
// (six spilled registers, outside the product loop) beat three without spills:
// 235 against 244 us.
//
// Tiles of 4 x 8 x 32 voxels; the next tile's loads are in flight during the
// products.  Partials per workgroup go to the workspace and are summed in a
// fixed order.

#include "cf_common.h"
#include "cf_kernels.h"
#include "conv_smallc4_halo.h"
#include "row_load.h"

#include <algorithm>

namespace cf {
namespace {

constexpr int TD = C4TD, TH = C4TH, TW = 32, HH = C4HH;
using Halo = C4Halo<TW, 8>;
constexpr int RP = Halo::NV * 8;           // halo row pitch (bytes)
constexpr int M = 108;                     // (tap, ci) rows

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x2_t tr4(const unsigned char *p) {
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)p));
}

template <bool DEF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void l1c4_wgrad_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ dp, const uint16_t *__restrict__ mask16, float alpha,
    float *__restrict__ part_w, float *__restrict__ part_b, SmallcParams p, C4Tiles tiles, int total_tiles) {
  // one array: halo | g, rne(alpha g) as [pd][ph][16 pw][16 ch] | mask [w-row][8-voxel
  // group]; the waves' sums take its place at the end
  constexpr int HB = C4ROWS * RP, GB = 256 * 16, SMEM = HB + 2 * GB + TD * TH * 64;
  constexpr int RB = 4 * (M + 1) * 16 * 4;
  static_assert(HB % 16 == 0, "16-byte rows");
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM > RB ? SMEM : RB];
  unsigned char *const halo = smem;
  uint4 *const gs = reinterpret_cast<uint4 *>(smem + HB);
  uint4 *const mks = reinterpret_cast<uint4 *>(smem + HB + 2 * GB);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, q = lane >> 4;
  // A: voxel 8 q + r / 4 (and 4 on), tap column min(r % 4, 2)
  const int kwl = (r & 3) < 2 ? (r & 3) : 2;
  const int aoff = (8 * q + (r >> 2) + kwl) * 8;
  // B: pooled voxel 4 q + r / 4, channels 4 (r % 4) ..
  const int goff = (4 * q + (r >> 2)) * 32 + 8 * (r & 3);
  const u32x4_t ones4 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, ones4);

  f32x4_t acc[9], acc_u = {0.f, 0.f, 0.f, 0.f}, acc_m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 9; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  Halo hl;
  hl.init(tid, p);
  u32x4_t xv[Halo::NL], dv, mv;
  auto load_tile = [&](int tile) {
    const C4Tile tl = c4_tile(tile, tiles, TW);
    const int n = tl.n, od0 = tl.d, oh0 = tl.h, ow0 = tl.w;
    hl.load(x, p, tl, xv);
    // pooled gradient: pooled voxel (tid >> 7, (tid >> 5) & 3, (tid >> 1) & 15), 8 channels
    dv = u32x4_t{0u, 0u, 0u, 0u};
    {
      const int pd_ = (od0 >> 1) + (tid >> 7), ph_ = (oh0 >> 1) + ((tid >> 5) & 3), pw_ = (ow0 >> 1) + ((tid >> 1) & 15);
      if (pd_ < p.pod && ph_ < p.poh && pw_ < p.pow_)
        dv = *reinterpret_cast<const u32x4_t *>(
            dp + ((((long long)n * p.pod + pd_) * p.poh + ph_) * p.pow_ + pw_) * 16 + 8 * (tid & 1));
    }
    // slope mask: thread tid < 128 loads 8 voxels (16 bytes) of w-row tid / 4; voxels
    // past the row pool into no window (their g is zero), so only the row is read
    mv = u32x4_t{0u, 0u, 0u, 0u};
    if (tid < 128) {
      const int row = tid >> 2;
      const int vd = od0 + row / TH, vh = oh0 + row % TH, vw = ow0 + 8 * (tid & 3);
      if (vd < p.od && vh < p.oh && vw < p.ow) {
        mv = load_mask8(mask16 + (((long long)n * p.od + vd) * p.oh + vh) * p.ow + vw, vw, p.ow);
      }
    }
  };

  // tiles in eight contiguous runs, one per XCD (workgroup b runs on XCD b % 8)
  const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, nwg = gridDim.x >> 3;
  const int per = (total_tiles + 7) >> 3;
  const int tend = min(total_tiles, (xcd + 1) * per);
  int tile = xcd * per + wg;
  if (tile < tend) load_tile(tile);
  for (; tile < tend; tile += nwg) {
#pragma unroll
    for (int k = 0; k < Halo::NL; ++k)
      if (tid + 256 * k < Halo::ITEMS)
        *reinterpret_cast<u32x4_t *>(halo + (hl.pk[k] & 63) * RP + (hl.pk[k] >> 8) * 16) = xv[k];
    gs[tid] = make_uint4(dv[0], dv[1], dv[2], dv[3]);
    uint32_t ga[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      ga[k] = f2bf2(alpha * __uint_as_float(dv[k] << 16), alpha * __uint_as_float(dv[k] & 0xffff0000u));
    gs[256 + tid] = make_uint4(ga[0], ga[1], ga[2], ga[3]);
    if (tid < 128) mks[tid] = make_uint4(mv[0], mv[1], mv[2], mv[3]);
    __syncthreads();
    if (tile + nwg < tend) load_tile(tile + nwg);

#pragma unroll 1
    for (int pp = 0; pp < 2; ++pp) {
      const int prow = wave + 4 * pp;  // pooled row (a, b) = (prow / 4, prow % 4)
      const int pa = prow >> 2, pb = prow & 3;
      const u32x2_t gq = tr4(smem + HB + prow * 512 + goff);
      const u32x2_t aq = tr4(smem + HB + GB + prow * 512 + goff);
      u32x4_t bu, ba;
      bu[0] = __builtin_amdgcn_perm(gq[0], gq[0], 0x01000100u);
      bu[1] = __builtin_amdgcn_perm(gq[0], gq[0], 0x03020302u);
      bu[2] = __builtin_amdgcn_perm(gq[1], gq[1], 0x01000100u);
      bu[3] = __builtin_amdgcn_perm(gq[1], gq[1], 0x03020302u);
      ba[0] = __builtin_amdgcn_perm(aq[0], aq[0], 0x01000100u);
      ba[1] = __builtin_amdgcn_perm(aq[0], aq[0], 0x03020302u);
      ba[2] = __builtin_amdgcn_perm(aq[1], aq[1], 0x01000100u);
      ba[3] = __builtin_amdgcn_perm(aq[1], aq[1], 0x03020302u);
      acc_u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8_t, bu), acc_u, 0, 0, 0);
      bf16x8_t bz[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = (2 * pa + (k >> 1)) * TH + 2 * pb + (k & 1);
        const uint4 mq = mks[row * 4 + q];
        const uint32_t mk[4] = {mq.x, mq.y, mq.z, mq.w};
        // mask dword d holds channel bits of voxels 2d (bits 0..15) and 2d+1 (16..31):
        // move bit r and bit 16+r to the two sign positions, spread each over its half
        typedef short v2i16_t __attribute__((ext_vector_type(2)));
        u32x4_t z, m;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t sg = __builtin_bit_cast(
              uint32_t, (v2i16_t)(__builtin_bit_cast(v2i16_t, mk[d] << (15 - r)) >> (v2i16_t){15, 15}));
          m[d] = bu[d] & sg;
          z[d] = m[d] | (ba[d] & ~sg);
        }
        acc_m = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8_t, m), acc_m, 0, 0, 0);
        bz[k] = __builtin_bit_cast(bf16x8_t, z);
      }
      const unsigned char *hb = halo + (2 * pa * HH + 2 * pb) * RP + aoff;
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const unsigned char *hr = hb + (a * HH + b) * RP;
          const u32x2_t lo = tr4(hr), hi = tr4(hr + 32);
          const u32x4_t av4 = {lo[0], lo[1], hi[0], hi[1]};
          const bf16x8_t av = __builtin_bit_cast(bf16x8_t, av4);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const int kd = a - i, kh = b - j;
              if (kd >= 0 && kd < 3 && kh >= 0 && kh < 3)
                acc[kd * 3 + kh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bz[2 * i + j], acc[kd * 3 + kh], 0, 0, 0);
            }
        }
    }
    __syncthreads();
  }

  // ---- combine the four waves: acc[k][e] = row (kernel row k, kw = q, ci = e), column r
  const float cu = 0.5f * alpha, cm = 0.125f * (1.f - alpha);
  float (*const red)[M + 1][16] = reinterpret_cast<float (*)[M + 1][16]>(smem);
  if (q < 3) {
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][(k * 3 + q) * 4 + e][r] = 0.125f * acc[k][e];
  } else {
    // four voxel rows share one product of ones with g
    red[wave][M][r] = cu * acc_u[0] + (alpha == 1.f ? 0.f : cm * acc_m[0]);
  }
  __syncthreads();
  // every wave looks at all 64 sums of db: the workgroup takes one way
  const bool by_def =
      DEF && (alpha > 1.f || __builtin_amdgcn_ballot_w64(!(fabsf(red[lane >> 4][M][lane & 15]) < __builtin_inff())));
  for (int i = tid; i < (M + 1) * 16; i += 256) {
    const int row = i >> 4, co = i & 15;
    const float v = red[0][row][co] + red[1][row][co] + red[2][row][co] + red[3][row][co];
    if (row < M) part_w[(long long)blockIdx.x * M * 16 + i] = v;
    else if (!by_def) part_b[(long long)blockIdx.x * 16 + co] = v;
  }
  if (by_def) {  // (uniform)
    float sb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // thread: the pooled voxel and channel half it loads in load_tile
    for (int t = xcd * per + wg; t < tend; t += nwg) {
      const C4Tile tl = c4_tile(t, tiles, TW);
      const int pd_ = (tl.d >> 1) + (tid >> 7), ph_ = (tl.h >> 1) + ((tid >> 5) & 3), pw_ = (tl.w >> 1) + ((tid >> 1) & 15);
      if (pd_ >= p.pod || ph_ >= p.poh || pw_ >= p.pow_) continue;
      const uint16_t *g =
          dp + ((((long long)tl.n * p.pod + pd_) * p.poh + ph_) * p.pow_ + pw_) * 16 + 8 * (tid & 1);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int vd = 2 * pd_ + (k >> 2), vh = 2 * ph_ + ((k >> 1) & 1), vw = 2 * pw_ + (k & 1);
        const uint32_t bits = mask16[(((long long)tl.n * p.od + vd) * p.oh + vh) * p.ow + vw] >> (8 * (tid & 1));
#pragma unroll
        for (int j = 0; j < 8; ++j) sb[j] += bf2f(g[j]) * 0.125f * ((bits >> j & 1u) ? 1.f : alpha);
      }
    }
    __syncthreads();  // every wave has read its sums
    float *const sums = reinterpret_cast<float *>(smem);  // [128 pooled voxels][16 channels]
#pragma unroll
    for (int j = 0; j < 8; ++j) sums[(tid >> 1) * 16 + 8 * (tid & 1) + j] = sb[j];
    __syncthreads();
    if (tid < 16) {
      float v = 0.f;
      for (int k = 0; k < 128; ++k) v += sums[k * 16 + tid];
      part_b[(long long)blockIdx.x * 16 + tid] = v;
    }
  }
}

// workgroups (each writes a 7 KB partial): four per compute unit stay resident
// (28 KB of LDS, at most 128 registers), a multiple of the eight XCDs
int c4_blocks(const ConvShape &s) {
  long long total;
  c4_tiles(s, TW, &total);
  return (int)std::min<long long>((total + 7) / 8 * 8, 4 * kNumCUs);
}

}  // namespace

bool l1c4_wgrad_supported(const ConvShape &s) {
  return s.dtype == DT_BF16 && l1c4_supported(s);
}

size_t l1c4_wgrad_workspace(const ConvShape &s) { return (size_t)c4_blocks(s) * (M + 1) * 16 * sizeof(float); }

hipError_t launch_l1c4_wgrad(const ConvShape &s, const void *x, const void *dp, const uint16_t *mask, float alpha,
                             float *dw, float *db, void *ws, hipStream_t st) {
  long long total;
  const C4Tiles tiles = c4_tiles(s, TW, &total);
  const int blocks = c4_blocks(s);
  float *pw = (float *)ws, *pb = pw + (size_t)blocks * M * 16;
  const bool def = alpha == 0.f || alpha > 1.f;
  hipLaunchKernelGGL((def ? l1c4_wgrad_kernel<true> : l1c4_wgrad_kernel<false>), dim3(blocks), dim3(256), 0, st,
                     (const uint16_t *)x, (const uint16_t *)dp, mask, alpha, pw, pb, c4_params(s), tiles, (int)total);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_sum_rows(pw, dw, blocks, M * 16, st);
  if (e != hipSuccess) return e;
  return launch_sum_rows(pb, db, blocks, 16, st);
}

}  // namespace cf
