// Shared by the kernels of the Fresnel stage (row, column, angular-spectrum and
// adjoint passes): launch geometry, the interpolated row of Eq. 5, the storage
// formats of H, and the dispatch over frame sizes.
//
// Index conventions: FFT position i carries original sample (i + N/2) mod N;
// the tables already hold (-1)^i' and the chirp, so both passes are plain
// positive-exponent DFTs and the output lands at natural (u, v).
#pragma once
#include "access.hpp"
#include "fft_engine.hpp"
#include "internal.hpp"
#include "split.hpp"

namespace ssoct {

// Tuning knobs (compile-time; the defaults are the tuned values)
#ifndef SSOCT_ROW_RPG
#define SSOCT_ROW_RPG 8          // rows per row group and workgroup iteration count
#endif
#ifndef SSOCT_ROW_PER_CU
#define SSOCT_ROW_PER_CU 2       // row passes: workgroups per CU a launch is split for
#endif
#ifndef SSOCT_ROW_WAVESYNC
#define SSOCT_ROW_WAVESYNC 1     // single-wave row groups exchange with wave-level ordering
#endif
#ifndef SSOCT_COL_MIN
#define SSOCT_COL_MIN 16         // minimum adjacent columns per column workgroup (128 B row segments)
#endif
#ifndef SSOCT_COL_PREFETCH
#define SSOCT_COL_PREFETCH 0     // load the next column tile while transforming the current one (always on
                                 // where the twiddles are in LDS, see SSOCT_COL_TWL)
#endif
#ifndef SSOCT_COL_TWL
#define SSOCT_COL_TWL 1          // column passes (Fresnel and angular-spectrum): twiddles in LDS where the
                                 // exchange buffer leaves room, and the next tile prefetched into registers
#endif
#ifndef SSOCT_COL_NT
#define SSOCT_COL_NT 1           // column pass: non-temporal stores of H
#endif

// Row pass geometry: GR groups of G = N/16 threads, each group owns rpg <= RPG
// consecutive rows (chosen per launch, row_rpg); a workgroup covers GR * rpg
// rows of one frame.  The kernels take rpg as a template argument SR for the
// launches that fill the chip (SR = 0: the kernel argument): with a run-time
// trip count the row loop is scheduled 2 % slower there.
template <int N>
struct RowCfg {
  static constexpr int G = FFTShape<N>::G;
  static constexpr int GR = (256 / G) < N ? (256 / G) : N;
  static constexpr int RPG = (N / GR) < SSOCT_ROW_RPG ? (N / GR) : SSOCT_ROW_RPG;
  static constexpr int ROWS = GR * RPG;                  // most rows per workgroup
  static constexpr int THREADS = GR * G;
  static constexpr bool WAVE = G <= 64 && SSOCT_ROW_WAVESYNC;  // a group lives inside one wavefront
};
// Column pass geometry: C adjacent columns (>= SSOCT_COL_MIN, so row segments
// are >= 64 B), at most 1024 threads
template <int N>
struct ColCfg {
  static constexpr int G = FFTShape<N>::G;
  static constexpr int C0 = 4096 / N;
  static constexpr int C1 = C0 < SSOCT_COL_MIN ? SSOCT_COL_MIN : (C0 > N ? N : C0);
  static constexpr int C = C1 * G > 1024 ? 1024 / G : C1;
  static constexpr int THREADS = C * G;
};
// Narrower tiles (C/2 and C/4 adjacent columns, for N >= 512) are tuning
// alternatives of the Fresnel column passes: fewer threads and less LDS per
// workgroup, so more workgroups per CU, at the price of shorter row segments.
template <int N>
struct ColTiles {
  static constexpr int C = ColCfg<N>::C;
  static constexpr bool ALT = N >= 512 && C >= 4;
  static constexpr int C2 = ALT ? C / 2 : C;
  static constexpr int C4 = ALT ? C / 4 : C;
};
// Columns per thread of the column passes.  At N = 2048 the exchange buffer
// holds 8 columns at most, and 64-byte row segments 16 KB apart run at half the
// rate of 128-byte ones (2.7 against 5.3 TB/s at N = 1024; 32-byte segments
// at half of that again).  There a thread of the default tile takes two
// adjacent columns (16-byte accesses, 128-byte segments per 8 threads) and
// transforms them one after the other through the same buffer: 100 -> 68 us per
// 4 frames (4.0 TB/s), without the next tile in registers.  The second column does
// not quite fit the 128 VGPRs of a thread of 1024: the default variant spills 27
// (112 bytes per lane; one column per thread none), with the Eq. 6 factor 88 (one
// column 44), in the second radix order, whose passes all have twiddles, 76 .. 121.
// Renders of T = 16 in the frame order, one column -> two: 761 -> 640 us, with the
// Eq. 6 factor 915 -> 826 us, in the second radix order 751 -> 771 us.
template <int N, int CT>
struct ColWide {
  static constexpr int W = N == 2048 && CT == ColCfg<N>::C ? 2 : 1;
};
// LDS of the column pass: the exchange buffer of CT columns, plus the twiddle
// table of radix order PL where the two fit in one CU's 160 KB (every N <= 1024;
// at N = 2048 the table without its repeated entries does, in the default order)
template <int N, int CT, int PL = 0>
struct ColLdsT {
  static constexpr int XB = FFTShape<N>::LDS * CT;
  static constexpr int FULL = TwPlan<N, PL>::SIZE > 0 ? TwPlan<N, PL>::SIZE : 1;
  static constexpr bool SMALL = PL == 0 && TwSmall<N>::OK && (XB + FULL) * 8 > 163840;
  static constexpr int TWN = SMALL ? TwSmall<N>::SIZE : FULL;
  static constexpr bool TWL = SSOCT_COL_TWL && (XB + TWN) * 8 <= 163840;
  // next tile prefetched into registers, where they do not hold a second column
  static constexpr bool PF = (TWL || SSOCT_COL_PREFETCH) && ColWide<N, CT>::W == 1;
  static constexpr int BYTES = (XB + (TWL ? TWN : 1)) * 8;
};
template <int N>
using ColLds = ColLdsT<N, ColCfg<N>::C>;

// Source rows y0 and y0 + 1 of Eq. 5 for one output row: thread j of a group
// holds columns [s N/4 + 4 j, s N/4 + 4 j + 4) for s = 0..3, so every load
// instruction of a group covers a contiguous N/2-byte span and the LDS stores
// of the y-lerped row are conflict free.
struct RowSrc {
  uint2 a[4], b[4];
};

template <int N>
__device__ __forceinline__ RowSrc load_rows(const uint16_t* __restrict__ I, int y0, int j) {
  const int y1 = y0 + 1 < N ? y0 + 1 : N - 1;
  const uint16_t* r0 = I + (size_t)y0 * N + 4 * j;
  const uint16_t* r1 = I + (size_t)y1 * N + 4 * j;
  RowSrc s;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s.a[q] = *reinterpret_cast<const uint2*>(r0 + q * (N / 4));
    s.b[q] = *reinterpret_cast<const uint2*>(r1 + q * (N / 4));
  }
  return s;
}

// y-lerp of the two source rows into rbuf (same column split as load_rows);
// the last thread also zeroes rbuf[N], the right tap of the last sample, which
// only occurs with weight 0 (s_t <= 1 keeps every position inside [0, N-1])
template <int N>
__device__ __forceinline__ void lerp_rows(const RowSrc& s, float fy, float* rbuf, int j) {
  if (j == N / 16 - 1) rbuf[N] = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t wa[2] = {s.a[q].x, s.a[q].y};
    const uint32_t wb[2] = {s.b[q].x, s.b[q].y};
    float out[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float a0 = (float)(wa[h] & 0xffffu), a1 = (float)(wa[h] >> 16);
      const float b0 = (float)(wb[h] & 0xffffu), b1 = (float)(wb[h] >> 16);
      out[2 * h] = a0 + fy * (b0 - a0);
      out[2 * h + 1] = a1 + fy * (b1 - a1);
    }
    *reinterpret_cast<float4*>(rbuf + q * (N / 4) + 4 * j) = make_float4(out[0], out[1], out[2], out[3]);
  }
}

// Aberration phase of one row as a quartic in x (cycles), from the per-row table
struct ARow {
  float p0, p1, p2, p3, p4;
};

template <bool ABERR>
__device__ __forceinline__ ARow load_arow(const float* __restrict__ apoly, int m) {
  ARow a{0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (ABERR) {
    const float4 lo = *reinterpret_cast<const float4*>(apoly + (size_t)m * APOLY_STRIDE);
    a = ARow{lo.x, lo.y, lo.z, lo.w, apoly[(size_t)m * APOLY_STRIDE + 4]};
  }
  return a;
}

// exp(2 pi i phase) of the aberration at FFT column n: Horner in FP32, the
// phase reduced to one cycle, then the hardware sine and cosine, which take
// their argument in cycles (measured on gfx950 over [-1/2, 1/2]: at most
// 1.3e-7 from the FP64 values)
template <int N>
__device__ __forceinline__ float2 aberr_factor(const ARow& a, int n) {
  constexpr float inv = 1.41421356237309505f / (float)N;   // rho = r / (N / sqrt 2)
  const float x = (float)(((n + N / 2) & (N - 1)) - N / 2) * inv;
  const float ph = fmaf(fmaf(fmaf(fmaf(a.p4, x, a.p3), x, a.p2), x, a.p1), x, a.p0);
  const float f = ph - rintf(ph);
  return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
}

// Row input z[m][n] of the DFT at FFT position n (x-lerp of the y-lerped row,
// times the separable chirp, dispersion, sign and optional aberration).
template <int N, bool ABERR>
__device__ __forceinline__ float2 row_input(const float* rbuf, const AxisTab& ct, float2 rowfac, const ARow& ar,
                                            int n) {
  const int x0 = ct.i0;
  const float r0 = rbuf[x0], r1 = rbuf[x0 + 1];   // rbuf[N] is a zero pad
  const float J = r0 + ct.f * (r1 - r0);
  float2 fac = cmul(ct.fac, rowfac);
  if constexpr (ABERR) fac = cmul(fac, aberr_factor<N>(ar, n));
  return make_float2(J * fac.x, J * fac.y);
}

template <int N>
struct RowLds {
  static constexpr int XS = (FFTShape<N>::LDS + 1) & ~1;  // row stride kept a multiple of 16 bytes
  AxisTab ctab[N];
  float2 xbuf[RowCfg<N>::GR][XS];   // exchange buffer; the y-lerped row (float4 stores) aliases its start
};

// stage the frame's column table in LDS (all threads)
template <int N>
__device__ __forceinline__ void stage_ctab(AxisTab* ctab, const AxisTab* __restrict__ src) {
  for (int i = threadIdx.x; i < N; i += RowCfg<N>::THREADS) ctab[i] = src[i];
}

// ------------------------------------------------------------------ H storage formats
template <int FMT, int NT = SSOCT_COL_NT>
__device__ __forceinline__ void store_h(void* __restrict__ H, long long idx, float2 val, float scale) {
  if constexpr (FMT == HF_F32) {
    st_once<NT>(reinterpret_cast<float2*>(H) + idx, val);
  } else {
    uint2 w;
    w.x = split_pack<FMT>(val.x * scale);
    w.y = split_pack<FMT>(val.y * scale);
    st_once<NT>(reinterpret_cast<uint2*>(H) + idx, w);
  }
}

// one pixel of an output format
template <int FMT>
struct HElem {
  using T = uint2;
};
template <>
struct HElem<HF_ABS> {
  using T = float;
};

// the same for W adjacent columns (W = 2: idx even, 16-byte stores), or their magnitudes
template <int FMT, int W, int NT>
__device__ __forceinline__ void store_h_cols(typename HElem<FMT>::T* __restrict__ H, uint32_t idx,
                                             const float2 (&val)[W], float scale) {
  if constexpr (FMT == HF_ABS) {
    float m[W];
#pragma unroll
    for (int w = 0; w < W; ++w) m[w] = sqrtf(val[w].x * val[w].x + val[w].y * val[w].y);
    if constexpr (W == 2)
      st_once<NT>(reinterpret_cast<float2*>(H + idx), make_float2(m[0], m[W - 1]));
    else
      st_once<NT>(H + idx, m[0]);
  } else if constexpr (W == 2) {
    uint4 q;
    if constexpr (FMT == HF_F32)
      q = make_uint4(__float_as_uint(val[0].x), __float_as_uint(val[0].y), __float_as_uint(val[1].x),
                     __float_as_uint(val[1].y));
    else
      q = make_uint4(split_pack<FMT>(val[0].x * scale), split_pack<FMT>(val[0].y * scale),
                     split_pack<FMT>(val[1].x * scale), split_pack<FMT>(val[1].y * scale));
    st_once<NT>(reinterpret_cast<uint4*>(H + idx), q);
  } else {
    store_h<FMT, NT>(H, idx, val[0], scale);
  }
}

// Rows per row group of a row pass over `planes` transforms of N rows: the
// largest of 8, 4, 2, 1 that still gives `per_cu` workgroups per CU, so that
// a launch of few rows spreads over the chip instead of running its rows one
// after another on a few CUs.  Such launches are bound by the latency of one row
// (load, transform, store), not by bandwidth: 16 frames at N = 512 take 16.6 us
// with 2 rows per group (512 workgroups) against 49 us with 8 (128), 32 frames
// at N = 256 13.2 against 27.8 us (adjoint 13.4 against 33.4 us).  Two
// workgroups per CU is where 8 rows at N = 1024 (16 frames) still win; 1, 4
// and 8 measured within 1 % of 2 over T = 30 .. 256, N = 64 .. 1024.
template <int N>
static int row_rpg(int planes, int cu, int per_cu) {
  using R = RowCfg<N>;
  int rpg = R::RPG;
  while (rpg > 1 && (long long)(N / (R::GR * rpg)) * planes < (long long)per_cu * cu) rpg /= 2;
  return rpg;
}

// persistent column workgroups: `req` (from the tuner) or 512 (two per CU of the 256 on MI355X)
inline int col_grid(int ntiles, int req) {
  const int g = req > 0 ? req : 512;
  return ntiles < g ? ntiles : g;
}

#define SSOCT_DISPATCH_N(N, CALL)        \
  switch (N) {                           \
    case 16: return CALL(16);            \
    case 32: return CALL(32);            \
    case 64: return CALL(64);            \
    case 128: return CALL(128);          \
    case 256: return CALL(256);          \
    case 512: return CALL(512);          \
    case 1024: return CALL(1024);        \
    case 2048: return CALL(2048);        \
    default: return hipErrorInvalidValue; \
  }

}  // namespace ssoct
