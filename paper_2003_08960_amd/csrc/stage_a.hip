// Row passes of the Fresnel stage (steps 1-2 of the flowchart, Fig. 3): chromatic
// rescale by linear interpolation (Eq. 5) fused with the chirp of Eq. 6 into the
// row DFT, and the row pass over depth-transformed frames (depth-first order).
//
// Persistent loops with register prefetch: a row group loads the source rows of
// its next output row while it transforms the current one.  The per-frame column
// table of Eq. 5/6 is staged in LDS once per row workgroup.
#include "stage.hpp"

namespace ssoct {

#ifndef SSOCT_ROWG_SPLIT
#define SSOCT_ROWG_SPLIT 2       // bin-pair row pass: below this many workgroups per CU the two transforms split
#endif
#ifndef SSOCT_ROW_NT
#define SSOCT_ROW_NT 0           // row pass: non-temporal stores of the intermediate
#endif
#ifndef SSOCT_ROWG_WPE
#define SSOCT_ROWG_WPE 2          // waves per SIMD the bin-pair row pass is held to (no aberration, no Eq. 6 factor)
#endif
#ifndef SSOCT_ROW_WAVES_PER_EU
#define SSOCT_ROW_WAVES_PER_EU 0  // > 0: ask the compiler to fit this many row-pass waves per SIMD
#endif
#if SSOCT_ROW_WAVES_PER_EU > 0
#define SSOCT_ROW_OCC __attribute__((amdgpu_waves_per_eu(SSOCT_ROW_WAVES_PER_EU)))
#else
#define SSOCT_ROW_OCC
#endif

// ------------------------------------------------------------------ forward row pass
template <int N, bool ABERR, bool EQ6, int SR>
__global__ __launch_bounds__(RowCfg<N>::THREADS) SSOCT_ROW_OCC void k_row_pass(
    const uint16_t* __restrict__ frames, int t0, const AxisTab* __restrict__ rows,
    const AxisTab* __restrict__ cols, const float2* __restrict__ tw, const float* __restrict__ apoly,
    const float2* __restrict__ outfac, float2* __restrict__ inter, int rpg_) {
  using S = FFTShape<N>;
  using R = RowCfg<N>;
  constexpr int G = S::G;
  const int rpg = SR ? SR : rpg_;
  const int wrows = R::GR * rpg;        // rows of this workgroup
  __shared__ RowLds<N> lds;
  __shared__ AxisTab rtab_s[R::ROWS];   // row table entries of this workgroup's rows
  // output factor of Eq. 6, read between the row's stores; kept in LDS up to
  // N = 1024 (at N = 2048 it would leave room for one workgroup per CU)
  constexpr bool OFS = EQ6 && N <= 1024;
  __shared__ float2 ofac_s[OFS ? N : 1];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int f = blockIdx.y;
  const int t = t0 + f;
  const int m0 = blockIdx.x * wrows + g * rpg;
  const uint16_t* I = frames + (size_t)t * N * N;
  const AxisTab* rtab = rows + (size_t)t * N;
  float* rbuf = reinterpret_cast<float*>(lds.xbuf[g]);
  // The first row's source loads, the twiddles and the table staging are in
  // flight together.  The twiddles stay in registers and the staging waits
  // complete their loads, so no twiddle load is outstanding inside the row
  // loop.  Inside the loop the next row's table entry comes from LDS: a
  // global load there would have to wait for the previous row's stores,
  // which the vector memory counter counts together with the loads.
  AxisTab rt = rtab[m0];
  RowSrc src = load_rows<N>(I, rt.i0, j);
  ARow an = load_arow<ABERR>(apoly, m0);
  const TwRegs<N> twr = load_tw_regs<N>(tw, j);
  stage_ctab<N>(lds.ctab, cols + (size_t)t * N);
  for (int i = threadIdx.x; i < wrows; i += R::THREADS) rtab_s[i] = rtab[blockIdx.x * wrows + i];
  if constexpr (OFS) {
    for (int i = threadIdx.x; i < N; i += R::THREADS) ofac_s[i] = outfac[i];
  }
  // Everything above has landed here (the first lerp needs it at once), so
  // the loop is entered with no load outstanding and its header, shared with
  // the back edge, does not wait for the stores of the previous row.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unchanged
  __syncthreads();  // column and row tables visible
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    const RowSrc cur = src;
    const AxisTab rc = rt;
    const ARow ar = an;
    if (i + 1 < rpg) {  // prefetch the next row of this group
      rt = rtab_s[g * rpg + i + 1];
      src = load_rows<N>(I, rt.i0, j);
      an = load_arow<ABERR>(apoly, m + 1);
    }
    exchange_sync<R::WAVE>();  // previous row's FFT reads are done
    lerp_rows<N>(cur, rc.f, rbuf, j);
    exchange_sync<R::WAVE>();
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int n = j + k * G;
      v[k] = row_input<N, ABERR>(rbuf, lds.ctab[n], rc.fac, ar, n);
    }
    fft_group_tw<N, +1, 1, R::WAVE>(v, j, lds.xbuf[g], twr);
    float2* dst = inter + ((size_t)f * N + m) * N;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int vv = j + out_offset<N>(e);
      float2 val = v[e];
      if constexpr (EQ6) val = cmul(val, OFS ? ofac_s[vv] : outfac[vv]);
      st_once<SSOCT_ROW_NT>(dst + vv, val);
    }
  }
}

// ------------------------------------------------------------------ bin-pair row pass (depth-first order)
// Row m of G_q (q = qa + f, FFT positions, from the depth DFT of the rescaled
// frames) times the frame-independent chirp, sign and optional aberration:
// DFT of fac G_q into chunk frame f and DFT of fac conj(G_q) into chunk frame
// Fh + f.  The column pass turns these into V[q] and V[T - q] (Eq. 6 is linear
// and its chirp does not depend on the frame when lambda_1 is used for every
// frame and no per-frame phase is applied).  Bin 0 of the stack holds the two
// real bins as one complex plane (G_0, G_T/2), so that every bin yields two
// transforms; its two are DFT of fac G_0 and of fac G_T/2.
//
// halves = 2 (small launches): the two transforms of a row go to two
// workgroups (blockIdx.y = h nb + f), so that twice as many wavefronts share a
// launch that leaves CUs idle; G is then read twice, from L2.
// Without the aberration factor the kernel fits two waves per SIMD; the
// compiler is held to that (with the Eq. 6 output factor it would otherwise
// take a few registers more and keep one).
template <int N, bool ABERR, bool EQ6, int SR>
__global__ __launch_bounds__(RowCfg<N>::THREADS)
__attribute__((amdgpu_waves_per_eu(ABERR ? 1 : (EQ6 ? 2 : SSOCT_ROWG_WPE)))) void k_row_pass_g(
    const float2* __restrict__ Gq, int qa, int nb, const AxisTab* __restrict__ rows0,
    const AxisTab* __restrict__ cols0, const float2* __restrict__ tw, const float* __restrict__ apoly,
    const float2* __restrict__ outfac, float2* __restrict__ inter, int Fh, int rpg_, int halves_) {
  using S = FFTShape<N>;
  using R = RowCfg<N>;
  constexpr int G = S::G;
  // column factors only (contiguous 8-byte entries: a 16-byte table entry read for its factor
  // alone would put two lanes on one LDS bank)
  __shared__ float2 cfac[N];
  __shared__ float2 xbuf[R::GR][RowLds<N>::XS];
  const int rpg = SR ? SR : rpg_;
  const int halves = SR ? 1 : halves_;
  const int wrows = R::GR * rpg;       // rows of this workgroup
  __shared__ float2 rfac_s[R::ROWS];   // row factors of this workgroup's rows
  constexpr bool OFS = EQ6 && N <= 1024;  // output factor of Eq. 6 in LDS, as in k_row_pass
  __shared__ float2 ofac_s[OFS ? N : 1];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int h0 = halves == 2 && (int)blockIdx.y >= nb ? 1 : 0;
  const int h1 = halves == 2 ? h0 + 1 : 2;
  const int f = blockIdx.y - h0 * nb;
  const int q = qa + f;
  const int m0 = blockIdx.x * wrows + g * rpg;
  float2 nxt[16];
  {
    const float2* src = Gq + ((size_t)q * N + m0) * N;
#pragma unroll
    for (int k = 0; k < 16; ++k) nxt[k] = ld_once<true>(src + j + k * G);
  }
  // as in k_row_pass: twiddles in registers, per-row table entries in LDS,
  // and no load outstanding when the loop is entered
  const TwRegs<N> twr = load_tw_regs<N>(tw, j);
  for (int i = threadIdx.x; i < N; i += R::THREADS) cfac[i] = cols0[i].fac;
  for (int i = threadIdx.x; i < wrows; i += R::THREADS) rfac_s[i] = rows0[blockIdx.x * wrows + i].fac;
  if constexpr (OFS) {
    for (int i = threadIdx.x; i < N; i += R::THREADS) ofac_s[i] = outfac[i];
  }
  ARow an = load_arow<ABERR>(apoly, m0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unchanged
  __syncthreads();  // column table and row factors visible
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    float2 gv[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) gv[k] = nxt[k];
    const ARow ar = an;
    if (i + 1 < rpg) {  // prefetch the next row of this group
      const float2* src = Gq + ((size_t)q * N + m + 1) * N;
#pragma unroll
      for (int k = 0; k < 16; ++k) nxt[k] = ld_once<true>(src + j + k * G);
      an = load_arow<ABERR>(apoly, m + 1);
    }
    const float2 rowfac = rfac_s[g * rpg + i];
#pragma unroll 1
    for (int h = h0; h < h1; ++h) {
      float2 v[16];
      auto factor = [&](int k) {
        const int n = j + k * G;
        float2 fac = cmul(cfac[n], rowfac);
        if constexpr (ABERR) fac = cmul(fac, aberr_factor<N>(ar, n));
        return fac;
      };
      if (q != 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = cmul(factor(k), h == 0 ? gv[k] : cconj(gv[k]));
      } else {   // the packed real bins
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = cscale(factor(k), h == 0 ? gv[k].x : gv[k].y);
      }
      exchange_sync<R::WAVE>();  // the previous transform's exchange reads are done
      fft_group_tw<N, +1, 1, R::WAVE>(v, j, xbuf[g], twr);
      float2* dst = inter + ((size_t)(h == 0 ? f : Fh + f) * N + m) * N;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int vv = j + out_offset<N>(e);
        float2 val = v[e];
        if constexpr (EQ6) val = cmul(val, OFS ? ofac_s[vv] : outfac[vv]);
        st_once<SSOCT_ROW_NT>(dst + vv, val);
      }
    }
  }
}

template <int N>
static hipError_t row_pass_n(int F, int t0, const uint16_t* frames, const AxisTab* rows, const AxisTab* cols,
                             const float2* tw, const float* apoly, const float2* outfac, float2* inter,
                             int cu, hipStream_t s) {
  using R = RowCfg<N>;
  const int rpg = row_rpg<N>(F, cu, SSOCT_ROW_PER_CU);
  dim3 grid(N / (R::GR * rpg), F), block(R::THREADS);
#define SSOCT_RP(A, E)                                                                                                 \
  do {                                                                                                                 \
    if (rpg == R::RPG)                                                                                                 \
      hipLaunchKernelGGL((k_row_pass<N, A, E, R::RPG>), grid, block, 0, s, frames, t0, rows, cols, tw, apoly, outfac,  \
                         inter, rpg);                                                                                  \
    else                                                                                                               \
      hipLaunchKernelGGL((k_row_pass<N, A, E, 0>), grid, block, 0, s, frames, t0, rows, cols, tw, apoly, outfac,       \
                         inter, rpg);                                                                                  \
  } while (0)
  if (apoly && outfac) SSOCT_RP(true, true);
  else if (apoly) SSOCT_RP(true, false);
  else if (outfac) SSOCT_RP(false, true);
  else SSOCT_RP(false, false);
#undef SSOCT_RP
  return hipGetLastError();
}

// Rows per group of the bin-pair row pass: `rpg` if it is one of 8, 4, 2, else
// 4 (8 rows measured slower at every launch size of the paper shape), halved
// while the launch would leave CUs without two workgroups; one row per group
// and still too few: the two transforms of each row in workgroups of their own.
template <int N>
static hipError_t row_pass_g_n(int nb, int qa, const float2* G, const AxisTab* rows0, const AxisTab* cols0,
                               const float2* tw, const float* apoly, const float2* outfac, float2* inter, int Fh,
                               int rpg, int cu, hipStream_t s) {
  using R = RowCfg<N>;
  int halves = 1;
  if (rpg != 8 && rpg != 4 && rpg != 2) {
    rpg = row_rpg<N>(nb, cu, 2);
    if (rpg > 4) rpg = 4;
    if (rpg == 1 && (long long)(N / R::GR) * nb < (long long)SSOCT_ROWG_SPLIT * cu) halves = 2;
  }
  if (rpg > R::RPG) rpg = R::RPG;
  dim3 grid(N / (R::GR * rpg), halves * nb), block(R::THREADS);
  constexpr int SR = R::RPG < 4 ? R::RPG : 4;
#define SSOCT_RG(A, E)                                                                                             \
  do {                                                                                                             \
    if (rpg == SR && halves == 1)                                                                                  \
      hipLaunchKernelGGL((k_row_pass_g<N, A, E, SR>), grid, block, 0, s, G, qa, nb, rows0, cols0, tw, apoly,       \
                         outfac, inter, Fh, rpg, halves);                                                          \
    else                                                                                                           \
      hipLaunchKernelGGL((k_row_pass_g<N, A, E, 0>), grid, block, 0, s, G, qa, nb, rows0, cols0, tw, apoly,        \
                         outfac, inter, Fh, rpg, halves);                                                          \
  } while (0)
  if (apoly && outfac) SSOCT_RG(true, true);
  else if (apoly) SSOCT_RG(true, false);
  else if (outfac) SSOCT_RG(false, true);
  else SSOCT_RG(false, false);
#undef SSOCT_RG
  return hipGetLastError();
}

hipError_t launch_row_pass(int N, int F, int t0, const uint16_t* frames, const AxisTab* rows, const AxisTab* cols,
                           const float2* tw, const float* apoly, const float2* outfac, float2* inter, int cu,
                           hipStream_t s) {
#define CALL(n) row_pass_n<n>(F, t0, frames, rows, cols, tw, apoly, outfac, inter, cu, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

hipError_t launch_row_pass_g(int N, int nb, int qa, const float2* G, const AxisTab* rows0,
                             const AxisTab* cols0, const float2* tw, const float* apoly, const float2* outfac,
                             float2* inter, int Fh, int rpg, int cu, hipStream_t s) {
#define CALL(n) row_pass_g_n<n>(nb, qa, G, rows0, cols0, tw, apoly, outfac, inter, Fh, rpg, cu, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

}  // namespace ssoct
