// Adjoint row pass of the gradient entry points.
#include "stage.hpp"

namespace ssoct {

#ifndef SSOCT_ADJ_PER_CU
#define SSOCT_ADJ_PER_CU 2       // adjoint row pass: workgroups per CU a launch is split for (as SSOCT_ROW_PER_CU)
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
  // Launches that fill the chip (SR) load the next row while the current one is computed and keep the
  // twiddles in LDS (at N = 2048 they would leave room for one workgroup per CU); with few rows per group
  // neither pays (64 frames of N = 256: 2.5 % of a gradient slower).
  constexpr bool PF = SR != 0;
  constexpr bool TWL = PF && N <= 1024;
  __shared__ RowLds<N> lds;
  __shared__ AxisTab rtab_s[PF ? R::ROWS : 1];
  __shared__ float2 twl[TWL && TwPlan<N>::SIZE > 0 ? TwPlan<N>::SIZE : 1];
  __shared__ double red[NW][N_MONO];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int f = blockIdx.y;
  const int t = t0 + f;
  const int rpg = SR ? SR : rpg_;
  const int wrows = R::GR * rpg;
  const int m0 = blockIdx.x * wrows + g * rpg;
  const uint16_t* I = frames + (size_t)t * N * N;
  const AxisTab* rtab = rows + (size_t)t * N;
  const float2* gin = inter + ((size_t)f * N + m0) * N + j;
  float* rbuf = reinterpret_cast<float*>(lds.xbuf[g]);
  // the first row's loads, the tables and the twiddles are in flight together
  AxisTab rt;
  float2 nx[16];
  RowSrc src;
  auto load_row = [&](int i) {
#pragma unroll
    for (int k = 0; k < 16; ++k) nx[k] = gin[(size_t)i * N + k * G];
    src = load_rows<N>(I, rt.i0, j);
  };
  if constexpr (PF) {
    rt = rtab[m0];
    load_row(0);
    for (int i = threadIdx.x; i < wrows; i += R::THREADS) rtab_s[i] = rtab[blockIdx.x * wrows + i];
  }
  stage_ctab<N>(lds.ctab, cols + (size_t)t * N);
  if constexpr (TWL) {
    for (int i = threadIdx.x; i < TwPlan<N>::SIZE; i += R::THREADS) twl[i] = tw[i];
  }
  const double inv = 1.4142135623730950488 / (double)N;
  const double xj = (double)j * inv;
  const int half = N >> 1;
  double acc[N_MONO];
#pragma unroll
  for (int k = 0; k < N_MONO; ++k) acc[k] = 0.0;
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    if constexpr (!PF) {
      rt = rtab[m];
      load_row(i);
    }
    const AxisTab rc = rt;
    const RowSrc cur = src;
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = nx[k];
    if (PF && i + 1 < rpg) {
      rt = rtab_s[g * rpg + i + 1];
      load_row(i + 1);
    }
    // the twiddles and the column table are read from LDS again for every row: kept over the loop they
    // would take 110 registers, and with the prefetched row the kernel would fall to one wave per SIMD
    int jc = j;
    asm volatile("" : "+v"(jc));
    exchange_sync<R::WAVE>();   // rbuf reads of the previous row are done
    fft_group_tw<N, -1, 1, R::WAVE>(v, j, lds.xbuf[g], TwMem<N>{TWL ? static_cast<const float2*>(twl) : tw, jc});
    float2 sc[ABERR ? 16 : 1];   // loads while the row is interpolated (before the transform they would not fit)
    if constexpr (ABERR) {
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[e] = screen[(size_t)m * N + j + out_offset<N>(e)];
    }
    exchange_sync<R::WAVE>();   // FFT reads of xbuf done before rbuf (aliased) is written
    lerp_rows<N>(cur, rc.f, rbuf, j);
    exchange_sync<R::WAVE>();
    // y is the same along the row: the row's sums of u x^a, then times y^b once per row (8 FP64 operations
    // per element for the five sums instead of 40 for the fifteen moments; the arithmetic, not the
    // 10 B/px, bounds this kernel: 63 -> 59 us per 64 frames of N = 512)
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int n = jc + out_offset<N>(e);
      float2 z = row_input<N, false>(rbuf, lds.ctab[n], rc.fac, ARow{}, n);
      if constexpr (ABERR) z = cmul(z, sc[e]);
      const float2 gg = v[e];
      const double u = (double)gg.x * (double)z.y - (double)gg.y * (double)z.x;  // Im(conj(g) z)
      // centred column: j + off, less N in the upper half (off alone decides the half: j < G)
      constexpr auto off = [](int k) { return out_offset<N>(k) < N / 2 ? out_offset<N>(k) : out_offset<N>(k) - N; };
      const double x = xj + (double)off(e) * inv;
      s0 += u;
      const double u1 = u * x;
      s1 += u1;
      s2 += u1 * x;
      const double u2 = u1 * x;
      s3 += u2 * x;
      const double u3 = u2 * x;
      s4 += u3 * x;
      if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    const double y = (double)(m < half ? m : m - N) * inv;
    const double y2 = y * y;
    acc[0] += s0;
    acc[1] += s1;
    acc[2] += s0 * y;
    acc[3] += s2;
    acc[4] += s1 * y;
    acc[5] += s0 * y2;
    acc[6] += s3;
    acc[7] += s2 * y;
    acc[8] += s1 * y2;
    acc[9] += s0 * (y2 * y);
    acc[10] += s4;
    acc[11] += s3 * y;
    acc[12] += s2 * y2;
    acc[13] += s1 * (y2 * y);
    acc[14] += s0 * (y2 * y2);
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
