// conv_igemm.hip -- general implicit-GEMM 3D convolution kernels for gfx950.
//
// Forward (Section III-C, Algorithm 1) and backward-data are both
// "output-stationary" contractions: every output voxel (GEMM row) is an inner
// product over (tap, channel) pairs (GEMM K) for every output channel (GEMM
// column).  Algorithm 1 blocks channels by the 16-lane SIMD width and output
// width by 28 registers; here the same contraction is tiled for MFMA:
// a 256-thread workgroup owns a BM x BN output tile, gathers the BM x BK
// slice of the (never materialised) im2col matrix and the BK x BN weight
// slice into LDS (double buffered), and four wave64s run
// v_mfma_f32_16x16x32_bf16 (bf16) or v_mfma_f32_16x16x4_f32 (fp32) on it
// with fp32 accumulation.
//
// Backward-data with stride s is split into s^3 parity classes of input
// voxels; in each class only the taps congruent to (i + pad) mod s reach an
// output voxel, so every class is a dense stride-one contraction over
// ceil(k/s)^3 taps (no multiply-by-zero work).  The weight slice is read
// transposed (W[t][ci][co] with co on the K axis).
//
// Backward-weights (Section III-C: a forward-like convolution with a large
// reduction and a small output, whose voxel slices accumulate privately and
// are then combined) is the contraction dW[(t,ci),co] = sum_p x~[p+t,ci]
// dz[p,co] over all output voxels p.  The voxel axis is split into fixed
// slices, one per workgroup column; each slice writes fp32 partials to the
// caller's workspace and a second kernel sums the partials in slice order
// (deterministic, no atomics).
//
// These kernels handle every shape (ragged tiles, any channel count); the
// vector path needs the gathered channel count to be a multiple of the
// 16-byte vector (8 bf16 / 4 fp32), otherwise a scalar gather is used.

#include "cf_common.h"
#include "cf_kernels.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>

namespace cf {
namespace {

template <int DT> struct Tile {
  // K depth of one LDS stage: 128 bytes of K per row in both dtypes.
  static constexpr int BK = DT == DT_BF16 ? 64 : 32;
  static constexpr int VEC = Store<DT>::VEC;
  static constexpr int LDK = BK + VEC;  // +16 B row padding against bank conflicts
};

// One MFMA pass over a BK-deep LDS stage: acc[fm][fn] += A_rows x B_cols.
// A_lds is [BM][LDK] (row-major, K contiguous), B_lds is [BN][LDK].
template <int DT, int FM, int FN>
__device__ __forceinline__ void mma_stage(const typename Store<DT>::T *__restrict__ a_lds,
                                          const typename Store<DT>::T *__restrict__ b_lds,
                                          int row0, int col0, int lane,
                                          f32x4_t (&acc)[FM][FN]) {
  constexpr int BK = Tile<DT>::BK;
  constexpr int LDK = Tile<DT>::LDK;
  const int r = lane & 15;
  const int q = lane >> 4;
  if constexpr (DT == DT_BF16) {
#pragma unroll
    for (int ks = 0; ks < BK; ks += 32) {
      bf16x8_t a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
        a[i] = *reinterpret_cast<const bf16x8_t *>(a_lds + (row0 + i * 16 + r) * LDK + ks + 8 * q);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        b[j] = *reinterpret_cast<const bf16x8_t *>(b_lds + (col0 + j * 16 + r) * LDK + ks + 8 * q);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      float a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = a_lds[(row0 + i * 16 + r) * LDK + ks + q];
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = b_lds[(col0 + j * 16 + r) * LDK + ks + q];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
}

// ---------------------------------------------------------------------------
// Forward / backward-data
// ---------------------------------------------------------------------------

struct IgemmParams {
  int nb;                      // batch
  int sd_, sh_, sw_, sc;       // gathered (source) tensor extent and channels
  int dd, dh, dw, dc;          // destination tensor extent and channels (= GEMM N)
  int jd, jh, jw;              // GEMM rows per dimension for this class
  int ostr_d, ostr_h, ostr_w;  // destination coordinate = j * ostr + orr
  int orr_d, orr_h, orr_w;
  int bstr_d, bstr_h, bstr_w;  // source base coordinate = j * bstr + bq
  int bq_d, bq_h, bq_w;
  int sgn;                     // source coordinate = base + sgn * u
  int ud, uh, uw;              // taps per dimension in this class
  int t0d, t0h, t0w;           // weight tap of u = 0
  int tsd, tsh, tsw;           // weight tap step per u
  int kh, kw;                  // kernel extents (weight indexing)
  int wci, wco;                // weight channel extents W[t][wci][wco]
  int ktot;                    // ud*uh*uw*sc
  int m;                       // nb*jd*jh*jw
};

template <int DT, int BM, int BN, int WM, int WN, bool VECA, bool DGRAD>
__global__ __launch_bounds__(256) void conv_igemm_kernel(const typename Store<DT>::T *__restrict__ src,
                                                         const typename Store<DT>::T *__restrict__ wt,
                                                         typename Store<DT>::T *__restrict__ dst,
                                                         IgemmParams p) {
  using T = typename Store<DT>::T;
  constexpr int BK = Tile<DT>::BK, VEC = Tile<DT>::VEC, LDK = Tile<DT>::LDK;
  constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  static_assert(WM * WN == 4, "four waves");
  static_assert(BM % 32 == 0 && BK / VEC == 8, "tile shape");
  __shared__ __attribute__((aligned(16))) T a_lds[2][BM * LDK];
  __shared__ __attribute__((aligned(16))) T b_lds[2][BN * LDK];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  if (m0 >= p.m) return;

  // ---- A gather setup ----------------------------------------------------
  // vector path: each thread owns one 16-byte K column (kv) and BM/32 rows.
  constexpr int AROWS = VECA ? BM / 32 : 1;
  int a_n[AROWS], a_bd[AROWS], a_bh[AROWS], a_bw[AROWS];
  const int kv = tid & 7;
  if constexpr (VECA) {
#pragma unroll
    for (int i = 0; i < AROWS; ++i) {
      int row = m0 + (tid >> 3) + 32 * i;
      if (row < p.m) {
        int jw_ = row % p.jw;
        int t = row / p.jw;
        int jh_ = t % p.jh;
        t /= p.jh;
        int jd_ = t % p.jd;
        a_n[i] = t / p.jd;
        a_bd[i] = jd_ * p.bstr_d + p.bq_d;
        a_bh[i] = jh_ * p.bstr_h + p.bq_h;
        a_bw[i] = jw_ * p.bstr_w + p.bq_w;
      } else {
        a_n[i] = -1;
        a_bd[i] = a_bh[i] = a_bw[i] = 0;
      }
    }
  }
  const int uhw = p.uh * p.uw;

  auto src_off = [&](int n, int cd, int ch, int cw, int c) -> long long {
    return ((((long long)n * p.sd_ + cd) * p.sh_ + ch) * p.sw_ + cw) * p.sc + c;
  };

  // registers holding the next stage
  uint4 a_reg[VECA ? AROWS : 1];
  T a_sreg[VECA ? 1 : BM * BK / 256];
  constexpr int BELEM = VECA ? 1 : BK * BN / 256;   // scalar weight path
  T b_reg[BELEM > 0 ? BELEM : 1];
  constexpr int BSLOTS = BN * (BK / VEC);            // 16-byte weight vectors per stage
  constexpr int NBV = VECA ? (BSLOTS + 255) / 256 : 1;
  uint4 b_vreg[NBV];

  auto load_stage = [&](int k0) {
    if constexpr (VECA) {
      int kk = k0 + kv * VEC;
      bool kin = kk < p.ktot;
      int u = kin ? kk / p.sc : 0;
      int c = kk - u * p.sc;
      int ud = u / uhw, uh = (u / p.uw) % p.uh, uw = u % p.uw;
#pragma unroll
      for (int i = 0; i < AROWS; ++i) {
        int cd = a_bd[i] + p.sgn * ud, ch = a_bh[i] + p.sgn * uh, cw = a_bw[i] + p.sgn * uw;
        bool ok = kin && a_n[i] >= 0 && (unsigned)cd < (unsigned)p.sd_ &&
                  (unsigned)ch < (unsigned)p.sh_ && (unsigned)cw < (unsigned)p.sw_;
        a_reg[i] = ok ? *reinterpret_cast<const uint4 *>(src + src_off(a_n[i], cd, ch, cw, c))
                      : make_uint4(0, 0, 0, 0);
      }
    } else {
      // scalar gather: element e = tid + 256*i -> (row = e / BK, k = e % BK)
#pragma unroll
      for (int i = 0; i < BM * BK / 256; ++i) {
        int e = tid + 256 * i;
        int row = m0 + e / BK;
        int kk = k0 + e % BK;
        T v = from_f32<DT>(0.f);
        if (row < p.m && kk < p.ktot) {
          int jw_ = row % p.jw;
          int t = row / p.jw;
          int jh_ = t % p.jh;
          t /= p.jh;
          int jd_ = t % p.jd;
          int n = t / p.jd;
          int u = kk / p.sc, c = kk - (kk / p.sc) * p.sc;
          int ud = u / uhw, uh = (u / p.uw) % p.uh, uw = u % p.uw;
          int cd = jd_ * p.bstr_d + p.bq_d + p.sgn * ud;
          int ch = jh_ * p.bstr_h + p.bq_h + p.sgn * uh;
          int cw = jw_ * p.bstr_w + p.bq_w + p.sgn * uw;
          if ((unsigned)cd < (unsigned)p.sd_ && (unsigned)ch < (unsigned)p.sh_ &&
              (unsigned)cw < (unsigned)p.sw_)
            v = src[src_off(n, cd, ch, cw, c)];
        }
        a_sreg[i] = v;
      }
    }
    if constexpr (VECA) {
      // weights, 16-byte vectors.  Forward: W[kk][n..n+VEC) (n contiguous).  Backward-data:
      // W[tap][n][c..c+VEC) (the K axis, output channels, contiguous).
#pragma unroll
      for (int i = 0; i < NBV; ++i) {
        const int slot = tid + 256 * i;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (slot < BSLOTS) {
          if constexpr (DGRAD) {
            const int kk0 = k0 + (slot & 7) * VEC, nn = n0 + (slot >> 3);
            if (kk0 < p.ktot && nn < p.dc) {
              int u = kk0 / p.sc, c0 = kk0 - u * p.sc;
              int ud = u / uhw, uh = (u / p.uw) % p.uh, uw = u % p.uw;
              int tap = ((p.t0d + p.tsd * ud) * p.kh + (p.t0h + p.tsh * uh)) * p.kw + (p.t0w + p.tsw * uw);
              v = *reinterpret_cast<const uint4 *>(wt + ((long long)tap * p.wci + nn) * p.wco + c0);
            }
          } else {
            const int kk = k0 + slot / (BN / VEC), nn0 = n0 + (slot % (BN / VEC)) * VEC;
            if (kk < p.ktot && nn0 < p.dc) v = *reinterpret_cast<const uint4 *>(wt + (long long)kk * p.wco + nn0);
          }
        }
        b_vreg[i] = v;
      }
    }
    // weights, scalar path: element e -> (k = e / BN, n = e % BN)
#pragma unroll
    for (int i = 0; i < (VECA ? 0 : BELEM); ++i) {
      int e = tid + 256 * i;
      int kk = k0 + e / BN;
      int nn = n0 + e % BN;
      T v = from_f32<DT>(0.f);
      if (kk < p.ktot && nn < p.dc) {
        int u = kk / p.sc, c = kk - (kk / p.sc) * p.sc;
        int ud = u / uhw, uh = (u / p.uw) % p.uh, uw = u % p.uw;
        int tap = ((p.t0d + p.tsd * ud) * p.kh + (p.t0h + p.tsh * uh)) * p.kw + (p.t0w + p.tsw * uw);
        long long off = DGRAD ? ((long long)tap * p.wci + nn) * p.wco + c
                              : ((long long)tap * p.wci + c) * p.wco + nn;
        v = wt[off];
      }
      b_reg[i] = v;
    }
  };

  auto store_stage = [&](int buf) {
    if constexpr (VECA) {
#pragma unroll
      for (int i = 0; i < AROWS; ++i)
        *reinterpret_cast<uint4 *>(&a_lds[buf][((tid >> 3) + 32 * i) * LDK + kv * VEC]) = a_reg[i];
    } else {
#pragma unroll
      for (int i = 0; i < BM * BK / 256; ++i) {
        int e = tid + 256 * i;
        a_lds[buf][(e / BK) * LDK + e % BK] = a_sreg[i];
      }
    }
    if constexpr (VECA) {
#pragma unroll
      for (int i = 0; i < NBV; ++i) {
        const int slot = tid + 256 * i;
        if (slot >= BSLOTS) continue;
        if constexpr (DGRAD) {
          *reinterpret_cast<uint4 *>(&b_lds[buf][(slot >> 3) * LDK + (slot & 7) * VEC]) = b_vreg[i];
        } else {
          Vec16<DT> v;
          v.u = b_vreg[i];
          const int kb = slot / (BN / VEC), nb0 = (slot % (BN / VEC)) * VEC;
#pragma unroll
          for (int j = 0; j < VEC; ++j) b_lds[buf][(nb0 + j) * LDK + kb] = v.e[j];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < BELEM; ++i) {
        int e = tid + 256 * i;
        b_lds[buf][(e % BN) * LDK + e / BN] = b_reg[i];
      }
    }
  };

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = (p.ktot + BK - 1) / BK;
  if (nk > 0) {
    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < nk) load_stage((kt + 1) * BK);
      mma_stage<DT, FM, FN>(a_lds[buf], b_lds[buf], wm * WTM, wn * WTN, lane, acc);
      if (kt + 1 < nk) store_stage(buf ^ 1);
      __syncthreads();
    }
  }

  // ---- epilogue: scatter the tile to the NDHWC destination ----------------
  const int q = lane >> 4, r = lane & 15;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int row = m0 + wm * WTM + i * 16 + 4 * q + j;
      if (row >= p.m) continue;
      int jw_ = row % p.jw;
      int t = row / p.jw;
      int jh_ = t % p.jh;
      t /= p.jh;
      int jd_ = t % p.jd;
      int n = t / p.jd;
      long long base = ((((long long)n * p.dd + jd_ * p.ostr_d + p.orr_d) * p.dh +
                         jh_ * p.ostr_h + p.orr_h) * p.dw + jw_ * p.ostr_w + p.orr_w) * p.dc;
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        int col = n0 + wn * WTN + f * 16 + r;
        if (col < p.dc) dst[base + col] = from_f32<DT>(acc[i][f][j]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Backward-weights: split reduction over output voxels + ordered sum
// ---------------------------------------------------------------------------

struct WgradParams {
  int nb, d, h, w, ci;
  int od, oh, ow, co;
  int kd, kh, kw;
  int sd, sh, sw, pd, ph, pw;
  int m;             // kd*kh*kw*ci (GEMM rows)
  long long pvox;    // nb*od*oh*ow (reduction length)
  long long chunk;   // voxels per slice, multiple of BK
};

template <int DT, int BM, int BN, int WM, int WN, bool VEC_OK>
__global__ __launch_bounds__(256) void conv_wgrad_kernel(const typename Store<DT>::T *__restrict__ x,
                                                         const typename Store<DT>::T *__restrict__ dz,
                                                         float *__restrict__ part, WgradParams p) {
  using T = typename Store<DT>::T;
  constexpr int BK = Tile<DT>::BK, VEC = Tile<DT>::VEC, LDK = Tile<DT>::LDK;
  constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  static_assert(WM * WN == 4, "four waves");
  static_assert(256 % BK == 0, "voxel lane mapping");
  __shared__ __attribute__((aligned(16))) T a_lds[2][BM * LDK];
  __shared__ __attribute__((aligned(16))) T b_lds[2][BN * LDK];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const long long pbeg = (long long)blockIdx.z * p.chunk;
  const long long pend = pbeg + p.chunk < p.pvox ? pbeg + p.chunk : p.pvox;
  const int pl = tid % BK;        // the voxel column this thread gathers
  const int rgrp = tid / BK;      // 0 .. 256/BK - 1
  constexpr int RSTEP = 256 / BK;
  const int taps_hw = p.kh * p.kw;

  constexpr int AV = VEC_OK ? VEC : 1;        // elements per gathered A item
  constexpr int AG = BM / AV, BG = BN / AV;   // row / column groups per stage
  constexpr int NA = (AG + RSTEP - 1) / RSTEP;  // A items per thread
  constexpr int NB = (BG + RSTEP - 1) / RSTEP;  // B items per thread
  union AItem { uint4 u; T e[VEC]; };
  AItem a_reg[NA], b_reg[NB];

  auto load_stage = [&](long long p0) {
    long long pv = p0 + pl;
    bool pin = pv < pend;
    int n = 0, bd = 0, bh = 0, bw = 0;
    long long dz_off = 0;
    if (pin) {
      long long t = pv;
      int ow_ = (int)(t % p.ow); t /= p.ow;
      int oh_ = (int)(t % p.oh); t /= p.oh;
      int od_ = (int)(t % p.od);
      n = (int)(t / p.od);
      bd = od_ * p.sd - p.pd;
      bh = oh_ * p.sh - p.ph;
      bw = ow_ * p.sw - p.pw;
      dz_off = pv * p.co;
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      int g = rgrp + RSTEP * i;
      int mrow = m0 + g * AV;
      int u = mrow / p.ci, c = mrow - (mrow / p.ci) * p.ci;
      int ud = u / taps_hw, uh = (u / p.kw) % p.kh, uw = u % p.kw;
      int cd = bd + ud, ch = bh + uh, cw = bw + uw;
      bool ok = pin && g < AG && mrow < p.m && (unsigned)cd < (unsigned)p.d && (unsigned)ch < (unsigned)p.h &&
                (unsigned)cw < (unsigned)p.w;
      long long off = ((((long long)n * p.d + cd) * p.h + ch) * p.w + cw) * p.ci + c;
      if constexpr (VEC_OK) {
        a_reg[i].u = ok ? *reinterpret_cast<const uint4 *>(x + off) : make_uint4(0, 0, 0, 0);
      } else {
        a_reg[i].e[0] = ok ? x[off] : from_f32<DT>(0.f);
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      int g = rgrp + RSTEP * i;
      int col = n0 + g * AV;
      bool ok = pin && g < BG && col < p.co;
      if constexpr (VEC_OK) {
        b_reg[i].u = ok ? *reinterpret_cast<const uint4 *>(dz + dz_off + col) : make_uint4(0, 0, 0, 0);
      } else {
        b_reg[i].e[0] = ok ? dz[dz_off + col] : from_f32<DT>(0.f);
      }
    }
  };

  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      int r0 = (rgrp + RSTEP * i) * AV;
      if (rgrp + RSTEP * i >= AG) continue;
#pragma unroll
      for (int j = 0; j < AV; ++j) a_lds[buf][(r0 + j) * LDK + pl] = a_reg[i].e[j];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      int c0 = (rgrp + RSTEP * i) * AV;
      if (rgrp + RSTEP * i >= BG) continue;
#pragma unroll
      for (int j = 0; j < AV; ++j) b_lds[buf][(c0 + j) * LDK + pl] = b_reg[i].e[j];
    }
  };

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = pend > pbeg ? (int)((pend - pbeg + BK - 1) / BK) : 0;
  if (nk > 0) {
    load_stage(pbeg);
    store_stage(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < nk) load_stage(pbeg + (long long)(kt + 1) * BK);
      mma_stage<DT, FM, FN>(a_lds[buf], b_lds[buf], wm * WTM, wn * WTN, lane, acc);
      if (kt + 1 < nk) store_stage(buf ^ 1);
      __syncthreads();
    }
  }

  float *out = part + (long long)blockIdx.z * p.m * p.co;
  const int q = lane >> 4, r = lane & 15;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int row = m0 + wm * WTM + i * 16 + 4 * q + j;
      if (row >= p.m) continue;
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        int col = n0 + wn * WTN + f * 16 + r;
        if (col < p.co) out[(long long)row * p.co + col] = acc[i][f][j];
      }
    }
}

// ---------------------------------------------------------------------------
// Host-side variant selection
// ---------------------------------------------------------------------------

template <int DT, int BM, int BN, int WM, int WN, bool DGRAD>
hipError_t launch_igemm(const IgemmParams &p, const void *src, const void *w, void *dst,
                        hipStream_t st) {
  using T = typename Store<DT>::T;
  dim3 grid((p.m + BM - 1) / BM, (p.dc + BN - 1) / BN, 1);
  // vector path: gathered channels and (forward) output channels multiples of the 16-byte vector
  if (p.sc % Store<DT>::VEC == 0 && (DGRAD || p.dc % Store<DT>::VEC == 0))
    hipLaunchKernelGGL((conv_igemm_kernel<DT, BM, BN, WM, WN, true, DGRAD>), grid, dim3(256), 0, st,
                       (const T *)src, (const T *)w, (T *)dst, p);
  else
    hipLaunchKernelGGL((conv_igemm_kernel<DT, BM, BN, WM, WN, false, DGRAD>), grid, dim3(256), 0, st,
                       (const T *)src, (const T *)w, (T *)dst, p);
  return hipGetLastError();
}

template <int DT, bool DGRAD>
hipError_t dispatch_igemm(const IgemmParams &p, const void *src, const void *w, void *dst,
                          hipStream_t st) {
  if (p.dc <= 16) return launch_igemm<DT, 128, 16, 4, 1, DGRAD>(p, src, w, dst, st);
  if (p.dc <= 32) return launch_igemm<DT, 128, 32, 4, 1, DGRAD>(p, src, w, dst, st);
  if (p.dc <= 64) return launch_igemm<DT, 128, 64, 2, 2, DGRAD>(p, src, w, dst, st);
  return launch_igemm<DT, 128, 128, 2, 2, DGRAD>(p, src, w, dst, st);
}

template <bool DGRAD>
hipError_t run_igemm(int dtype, const IgemmParams &p, const void *src, const void *w, void *dst,
                     hipStream_t st) {
  if (p.m <= 0) return hipSuccess;
  return dtype == DT_BF16 ? dispatch_igemm<DT_BF16, DGRAD>(p, src, w, dst, st)
                          : dispatch_igemm<DT_F32, DGRAD>(p, src, w, dst, st);
}

struct WgradPlan {
  int bm, bn;
  long long chunk;
  int nsplit;
};

WgradPlan plan_wgrad(const ConvShape &s) {
  WgradPlan pl;
  const int m = s.kd * s.kh * s.kw * s.ci;
  pl.bm = 64;
  pl.bn = s.co <= 16 ? 16 : (s.co <= 32 ? 32 : 64);
  const int bk = s.dtype == DT_BF16 ? Tile<DT_BF16>::BK : Tile<DT_F32>::BK;
  const long long pvox = (long long)s.n * s.od * s.oh * s.ow;
  const long long tiles = (long long)((m + pl.bm - 1) / pl.bm) * ((s.co + pl.bn - 1) / pl.bn);
  // aim for ~2048 workgroups, but give each slice at least 4 stages of work
  long long want = std::max(1LL, 2048 / std::max(1LL, tiles));
  long long chunk = (pvox + want - 1) / want;
  chunk = std::max<long long>(chunk, 4LL * bk);
  chunk = (chunk + bk - 1) / bk * bk;
  pl.chunk = chunk;
  pl.nsplit = (int)((pvox + chunk - 1) / chunk);
  if (pl.nsplit < 1) pl.nsplit = 1;
  return pl;
}

template <int DT, int BM, int BN, int WM, int WN>
hipError_t launch_wgrad_t(const WgradParams &p, int nsplit, const void *x, const void *dz,
                          float *part, hipStream_t st) {
  using T = typename Store<DT>::T;
  dim3 grid((p.m + BM - 1) / BM, (p.co + BN - 1) / BN, nsplit);
  constexpr int V = Store<DT>::VEC;
  if (p.ci % V == 0 && p.co % V == 0)
    hipLaunchKernelGGL((conv_wgrad_kernel<DT, BM, BN, WM, WN, true>), grid, dim3(256), 0, st,
                       (const T *)x, (const T *)dz, part, p);
  else
    hipLaunchKernelGGL((conv_wgrad_kernel<DT, BM, BN, WM, WN, false>), grid, dim3(256), 0, st,
                       (const T *)x, (const T *)dz, part, p);
  return hipGetLastError();
}

template <int DT>
hipError_t dispatch_wgrad(const WgradPlan &pl, const WgradParams &p, const void *x, const void *dz,
                          float *part, hipStream_t st) {
  if (pl.bn == 16) return launch_wgrad_t<DT, 64, 16, 4, 1>(p, pl.nsplit, x, dz, part, st);
  if (pl.bn == 32) return launch_wgrad_t<DT, 64, 32, 2, 2>(p, pl.nsplit, x, dz, part, st);
  return launch_wgrad_t<DT, 64, 64, 2, 2>(p, pl.nsplit, x, dz, part, st);
}

}  // namespace

// CF_CONV_KERNEL=igemm keeps forward and backward-data on the generic kernel,
// CF_CONV_KERNEL=c4 the fp32 four-channel forward on its own (tests compare the
// specialised fp32 kernels with the generic one this way)
static bool kernel_forced(const char *name) {
  const char *e = getenv("CF_CONV_KERNEL");
  return e && !strcmp(e, name);
}

static bool igemm_forced() { return kernel_forced("igemm"); }

// Four input channels in fp32 (the same bits from both kernels): a wave of the
// halo kernel goes through its 4 x 8 x 32 tile alone, 2.3 us for every eight voxels of
// a row, while the generic kernel takes 10 us up to 2^15 voxels (one round of its
// workgroups) and 13 us and more from there on.  So rows of up to 16 voxels run the
// halo kernel at any size (16^3 9.9 -> 8.0 us), longer ones past 2^15 voxels (32^3:
// 10.3 us generic, 12.9 halo; 32 x 32 x 36 13.2 and 13.0; 32 x 32 x 91 18.0 and 13.5).
static bool l1c4_fwd_taken(const ConvShape &s) {
  if (!l1c4_supported(s) || igemm_forced()) return false;
  return s.dtype == DT_BF16 || s.ow <= 16 || (long long)s.n * s.od * s.oh * s.ow > (1 << 15) || kernel_forced("c4");
}

hipError_t launch_conv_fwd(const ConvShape &s, const void *x, const void *w, void *z,
                           hipStream_t st) {
  // four input channels: operand fragments of whole voxels
  if (l1c4_fwd_taken(s)) return launch_conv_fwd_l1c4(s, x, w, nullptr, 0.f, z, nullptr, false, st);
  // few input channels: the direct halo kernel (one im2col gather per MFMA tile)
  if (smallc_supported(s, false))
    return launch_conv_fwd_smallc(s, x, w, nullptr, 0.f, z, nullptr, false, st);
  // 16 -> 32 channels, stride 1: halo-tiled MFMA kernel with weights resident in LDS
  if (c16_fwd_supported(s)) return launch_conv_fwd_c16(s, x, w, nullptr, 0.f, z, nullptr, 0, st);
  // many channels, bf16: waves split the taps, fragments gathered straight into registers
  if (direct_supported(s, true)) return launch_conv_fwd_direct(s, x, w, nullptr, 0.f, z, nullptr, false, st);
  // fp32 with 16k input channels: register-streaming fp32 MFMA kernel
  if (f32conv_supported(s, true) && !igemm_forced())
    return launch_conv_fwd_f32(s, (const float *)x, (const float *)w, nullptr, 0.f, (float *)z, nullptr, 0, st);
  IgemmParams p{};
  p.nb = s.n;
  p.sd_ = s.d; p.sh_ = s.h; p.sw_ = s.w; p.sc = s.ci;
  p.dd = s.od; p.dh = s.oh; p.dw = s.ow; p.dc = s.co;
  p.jd = s.od; p.jh = s.oh; p.jw = s.ow;
  p.ostr_d = p.ostr_h = p.ostr_w = 1;
  p.orr_d = p.orr_h = p.orr_w = 0;
  p.bstr_d = s.sd; p.bstr_h = s.sh; p.bstr_w = s.sw;
  p.bq_d = -s.pd; p.bq_h = -s.ph; p.bq_w = -s.pw;
  p.sgn = 1;
  p.ud = s.kd; p.uh = s.kh; p.uw = s.kw;
  p.t0d = p.t0h = p.t0w = 0;
  p.tsd = p.tsh = p.tsw = 1;
  p.kh = s.kh; p.kw = s.kw;
  p.wci = s.ci; p.wco = s.co;
  p.ktot = s.kd * s.kh * s.kw * s.ci;
  p.m = s.n * s.od * s.oh * s.ow;
  return run_igemm<false>(s.dtype, p, x, w, z, st);
}

hipError_t launch_conv_bwd_data(const ConvShape &s, const void *dz, const void *w, void *dx,
                                hipStream_t st) {
  if (c16_bwd_supported(s)) return launch_conv_bwd_data_c16(s, dz, nullptr, w, 0.f, dx, false, st);
  if (direct_supported(s, false)) return launch_conv_bwd_data_direct(s, dz, w, dx, st);
  if (f32conv_supported(s, false) && !igemm_forced())
    return launch_conv_bwd_data_f32(s, (const float *)dz, (const float *)w, (float *)dx, st);
  // one launch per parity class (r_d, r_h, r_w) of input voxels
  for (int rd = 0; rd < s.sd; ++rd)
    for (int rh = 0; rh < s.sh; ++rh)
      for (int rw = 0; rw < s.sw; ++rw) {
        IgemmParams p{};
        p.nb = s.n;
        p.sd_ = s.od; p.sh_ = s.oh; p.sw_ = s.ow; p.sc = s.co;
        p.dd = s.d; p.dh = s.h; p.dw = s.w; p.dc = s.ci;
        const int r[3] = {rd, rh, rw};
        const int ext[3] = {s.d, s.h, s.w};
        const int str[3] = {s.sd, s.sh, s.sw};
        const int pad[3] = {s.pd, s.ph, s.pw};
        const int ks[3] = {s.kd, s.kh, s.kw};
        int J[3], U[3], T0[3], Q[3];
        for (int a = 0; a < 3; ++a) {
          J[a] = ext[a] > r[a] ? (ext[a] - r[a] + str[a] - 1) / str[a] : 0;
          T0[a] = (r[a] + pad[a]) % str[a];
          U[a] = T0[a] < ks[a] ? (ks[a] - T0[a] + str[a] - 1) / str[a] : 0;
          Q[a] = (r[a] + pad[a] - T0[a]) / str[a];
        }
        p.jd = J[0]; p.jh = J[1]; p.jw = J[2];
        p.ostr_d = s.sd; p.ostr_h = s.sh; p.ostr_w = s.sw;
        p.orr_d = rd; p.orr_h = rh; p.orr_w = rw;
        p.bstr_d = p.bstr_h = p.bstr_w = 1;
        p.bq_d = Q[0]; p.bq_h = Q[1]; p.bq_w = Q[2];
        p.sgn = -1;
        p.ud = U[0]; p.uh = U[1]; p.uw = U[2];
        p.t0d = T0[0]; p.t0h = T0[1]; p.t0w = T0[2];
        p.tsd = s.sd; p.tsh = s.sh; p.tsw = s.sw;
        p.kh = s.kh; p.kw = s.kw;
        p.wci = s.ci; p.wco = s.co;
        p.ktot = U[0] * U[1] * U[2] * s.co;
        p.m = s.n * J[0] * J[1] * J[2];
        if (p.uh == 0) p.uh = 1;  // avoid division by zero in the decode; ktot is 0 then
        if (p.uw == 0) p.uw = 1;
        hipError_t e = run_igemm<true>(s.dtype, p, dz, w, dx, st);
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

// The generic tiled weight-gradient kernel serves what neither the 16 -> 32
// kernel nor the deep-layer kernel covers; CF_WGRAD_KERNEL=igemm forces it
// for the deep layers (tests compare the two).
static bool use_direct_wgrad(const ConvShape &s) {
  const char *e = getenv("CF_WGRAD_KERNEL");
  if (e && !strcmp(e, "igemm")) return false;
  return direct_wgrad_supported(s);
}

// the single-channel first layer (bf16): CF_WGRAD_KERNEL=igemm forces the generic kernel
// fp32 with 16k channels: CF_WGRAD_KERNEL=igemm forces the generic kernel
static bool use_f32_wgrad(const ConvShape &s) {
  const char *e = getenv("CF_WGRAD_KERNEL");
  if (e && !strcmp(e, "igemm")) return false;
  return f32wgrad_supported(s);
}

static bool use_l1_wgrad(const ConvShape &s) {
  const char *e = getenv("CF_WGRAD_KERNEL");
  if (e && !strcmp(e, "igemm")) return false;
  return smallc_wgrad_dz_supported(s);
}

size_t conv_bwd_weight_workspace(const ConvShape &s) {
  if (use_l1_wgrad(s)) return smallc_wgrad_dz_workspace(s);
  if (c16_wgrad_supported(s)) return c16_wgrad_workspace(s);
  if (use_direct_wgrad(s)) return direct_wgrad_workspace(s, false);
  if (use_f32_wgrad(s)) return f32wgrad_workspace(s, 0);
  WgradPlan pl = plan_wgrad(s);
  return (size_t)pl.nsplit * s.kd * s.kh * s.kw * s.ci * s.co * sizeof(float);
}

hipError_t launch_conv_bwd_weight(const ConvShape &s, const void *x, const void *dz, float *dw,
                                  void *ws, hipStream_t st) {
  if (use_l1_wgrad(s)) return launch_smallc_wgrad_dz(s, x, dz, dw, ws, st);
  if (c16_wgrad_supported(s))
    return launch_conv_bwd_weight_c16(s, x, dz, nullptr, 0.f, dw, nullptr, ws, false, nullptr, st);
  if (use_direct_wgrad(s))
    return launch_conv_bwd_weight_direct(s, x, dz, nullptr, DWG_DZ, 0.f, dw, nullptr, ws, st);
  if (use_f32_wgrad(s))
    return launch_conv_bwd_weight_f32(s, (const float *)x, (const float *)dz, nullptr, 0.f, dw, nullptr, ws, 0,
                                      nullptr, st);
  WgradPlan pl = plan_wgrad(s);
  WgradParams p{};
  p.nb = s.n; p.d = s.d; p.h = s.h; p.w = s.w; p.ci = s.ci;
  p.od = s.od; p.oh = s.oh; p.ow = s.ow; p.co = s.co;
  p.kd = s.kd; p.kh = s.kh; p.kw = s.kw;
  p.sd = s.sd; p.sh = s.sh; p.sw = s.sw; p.pd = s.pd; p.ph = s.ph; p.pw = s.pw;
  p.m = s.kd * s.kh * s.kw * s.ci;
  p.pvox = (long long)s.n * s.od * s.oh * s.ow;
  p.chunk = pl.chunk;
  float *part = (float *)ws;
  hipError_t e = s.dtype == DT_BF16 ? dispatch_wgrad<DT_BF16>(pl, p, x, dz, part, st)
                                    : dispatch_wgrad<DT_F32>(pl, p, x, dz, part, st);
  if (e != hipSuccess) return e;
  return launch_sum_rows(part, dw, pl.nsplit, p.m * p.co, st);
}

// weight and data gradients from one stored dz: the fp32 register-streamed
// kernels share one launch (launch_conv_bwd_f32); every other path runs the
// two dispatchers above in sequence
hipError_t launch_conv_bwd(const ConvShape &s, const void *x, const void *dz, const void *w, float *dw, void *dx,
                           void *ws, hipStream_t st) {
  const bool wf32 = !use_l1_wgrad(s) && !c16_wgrad_supported(s) && !use_direct_wgrad(s) && use_f32_wgrad(s);
  const bool df32 = !c16_bwd_supported(s) && !direct_supported(s, false) && f32conv_supported(s, false) &&
                    !igemm_forced();
  if (wf32 && df32)
    return launch_conv_bwd_f32(s, (const float *)x, (const float *)dz, (const float *)w, dw, (float *)dx, ws, st);
  hipError_t e = launch_conv_bwd_weight(s, x, dz, dw, ws, st);
  if (e != hipSuccess) return e;
  return launch_conv_bwd_data(s, dz, w, dx, st);
}

}  // namespace cf
