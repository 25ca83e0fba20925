// Adjoint row pass of the gradient entry points.
#include "stage.hpp"

namespace ssoct {

#ifndef SSOCT_ADJ_PER_CU
#define SSOCT_ADJ_PER_CU 2       // the same for the adjoint row pass
#endif

// ------------------------------------------------------------------ adjoint row pass + moments
// g[m][n] = DFT^-_v inter[f][m][v]; u = Im(conj(g) z) with z recomputed as in
// the forward row pass; per-(frame, workgroup) FP64 moments sum u x^a y^b
// (a + b <= 4) at the original sample (x, y) = (c_n', c_m') sqrt(2) / N.
template <int N, bool ABERR, int SR>
__global__ __launch_bounds__(RowCfg<N>::THREADS) void k_row_pass_adj(
    const uint16_t* __restrict__ frames, int t0, const AxisTab* __restrict__ rows,
    const AxisTab* __restrict__ cols, const float2* __restrict__ tw, const float2* __restrict__ screen,
    const float2* __restrict__ inter, double* __restrict__ partials, int rpg_) {
  using S = FFTShape<N>;
  using R = RowCfg<N>;
  constexpr int G = S::G;
  constexpr int NW = (R::THREADS + 63) / 64;
  constexpr int WIDTH = R::THREADS < 64 ? R::THREADS : 64;  // lanes that exist in a wave
  __shared__ RowLds<N> lds;
  __shared__ double red[NW][N_MONO];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int f = blockIdx.y;
  const int t = t0 + f;
  const int rpg = SR ? SR : rpg_;
  const int m0 = (blockIdx.x * R::GR + g) * rpg;
  const uint16_t* I = frames + (size_t)t * N * N;
  const AxisTab* rtab = rows + (size_t)t * N;
  float* rbuf = reinterpret_cast<float*>(lds.xbuf[g]);
  stage_ctab<N>(lds.ctab, cols + (size_t)t * N);
  const double inv = 1.4142135623730950488 / (double)N;
  const int half = N >> 1;
  double acc[N_MONO];
#pragma unroll
  for (int k = 0; k < N_MONO; ++k) acc[k] = 0.0;
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    const AxisTab rc = rtab[m];
    const RowSrc cur = load_rows<N>(I, rc.i0, j);
    const float2* srow_ab = ABERR ? screen + (size_t)m * N : nullptr;
    const float2* srow = inter + ((size_t)f * N + m) * N;
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = srow[j + k * G];
    fft_group<N, -1, 1, R::WAVE>(v, j, lds.xbuf[g], tw);
    exchange_sync<R::WAVE>();   // FFT reads of xbuf done before rbuf (aliased) is written
    lerp_rows<N>(cur, rc.f, rbuf, j);
    exchange_sync<R::WAVE>();
    const double y = (double)(m < half ? m : m - N) * inv;
    const double y2 = y * y;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int n = j + out_offset<N>(e);
      float2 z = row_input<N, false>(rbuf, lds.ctab[n], rc.fac, ARow{}, n);
      if constexpr (ABERR) z = cmul(z, srow_ab[n]);
      const float2 gg = v[e];
      const double u = (double)gg.x * (double)z.y - (double)gg.y * (double)z.x;  // Im(conj(g) z)
      const double x = (double)(n < half ? n : n - N) * inv;
      const double x2 = x * x;
      const double ux = u * x, uy = u * y;
      acc[0] += u;
      acc[1] += ux;
      acc[2] += uy;
      acc[3] += ux * x;
      acc[4] += ux * y;
      acc[5] += uy * y;
      acc[6] += ux * x2;
      acc[7] += ux * x * y;
      acc[8] += ux * y2;
      acc[9] += uy * y2;
      acc[10] += ux * x * x2;
      acc[11] += ux * x2 * y;
      acc[12] += ux * x * y2;
      acc[13] += ux * y2 * y;
      acc[14] += uy * y * y2;
    }
    exchange_sync<R::WAVE>();   // rbuf reads done before the next FFT writes xbuf
  }
  // wave reduction, then across waves in fixed order
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N_MONO; ++k) {
    double a = acc[k];
    for (int o = WIDTH / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, WIDTH);
    acc[k] = a;
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < N_MONO; ++k) red[wv][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x < N_MONO) {
    double s = 0.0;
    for (int w = 0; w < NW; ++w) s += red[w][threadIdx.x];
    partials[((size_t)t * gridDim.x + blockIdx.x) * N_MONO + threadIdx.x] = s;
  }
}

template <int N>
static hipError_t row_pass_adj_n(int F, int t0, const uint16_t* frames, const AxisTab* rows, const AxisTab* cols,
                                 const float2* tw, const float2* screen, const float2* inter, double* partials,
                                 int nblk, hipStream_t s) {
  using R = RowCfg<N>;
  const int rpg = N / (R::GR * nblk);
  if (nblk < 1 || rpg < 1 || rpg > R::RPG || R::GR * rpg * nblk != N) return hipErrorInvalidValue;
  dim3 grid(nblk, F), block(R::THREADS);
#define SSOCT_RA(A, SR)                                                                                              \
  hipLaunchKernelGGL((k_row_pass_adj<N, A, SR>), grid, block, 0, s, frames, t0, rows, cols, tw, screen, inter, partials, \
                     rpg)
  if (screen) { if (rpg == R::RPG) SSOCT_RA(true, R::RPG); else SSOCT_RA(true, 0); }
  else { if (rpg == R::RPG) SSOCT_RA(false, R::RPG); else SSOCT_RA(false, 0); }
#undef SSOCT_RA
  return hipGetLastError();
}

hipError_t launch_row_pass_adj(int N, int F, int t0, const uint16_t* frames, const AxisTab* rows,
                               const AxisTab* cols, const float2* tw, const float2* screen, const float2* inter,
                               double* partials, int nblk, hipStream_t s) {
#define CALL(n) row_pass_adj_n<n>(F, t0, frames, rows, cols, tw, screen, inter, partials, nblk, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

template <int N>
static int row_adj_blocks_n(int F, int cu) {
  using R = RowCfg<N>;
  return F > 0 ? N / (R::GR * row_rpg<N>(F, cu, SSOCT_ADJ_PER_CU)) : N / R::GR;
}

int row_adj_blocks(int N, int F, int cu) {
  switch (N) {
    case 16: return row_adj_blocks_n<16>(F, cu);
    case 32: return row_adj_blocks_n<32>(F, cu);
    case 64: return row_adj_blocks_n<64>(F, cu);
    case 128: return row_adj_blocks_n<128>(F, cu);
    case 256: return row_adj_blocks_n<256>(F, cu);
    case 512: return row_adj_blocks_n<512>(F, cu);
    case 1024: return row_adj_blocks_n<1024>(F, cu);
    case 2048: return row_adj_blocks_n<2048>(F, cu);
    default: return 0;
  }
}

}  // namespace ssoct
