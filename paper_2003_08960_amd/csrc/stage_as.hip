// Angular-spectrum propagation: row, column and inverse row passes.
#include "stage.hpp"

namespace ssoct {

#ifndef SSOCT_AS_XCD
#define SSOCT_AS_XCD 1           // transfer-function column pass: contiguous runs of tiles per XCD
#endif
#ifndef SSOCT_AS_GROUP
#define SSOCT_AS_GROUP 0         // > 0: phase evaluations scheduled in groups of this many
#endif
#ifndef SSOCT_AS_PF
#define SSOCT_AS_PF 1            // 1: transfer-function column pass loads its next tile while transforming
#endif
#ifndef SSOCT_AS_WPE
#define SSOCT_AS_WPE 0           // > 0: waves per SIMD the transfer-function column pass is compiled for
#endif
#if SSOCT_AS_WPE > 0
#define SSOCT_AS_OCC __attribute__((amdgpu_waves_per_eu(SSOCT_AS_WPE)))
#else
#define SSOCT_AS_OCC
#endif
#ifndef SSOCT_AS_THREADS
#define SSOCT_AS_THREADS 256     // transfer-function column pass: at most this many threads per workgroup
#endif

// ------------------------------------------------------------------ angular-spectrum passes
// Propagation of the sensor field by the angular spectrum (no rescale, no
// chirp, plain uncentred DFTs; pixel and frequency indices both natural):
//   pass 1 (k_as_row_fwd): DFT^- of the u16 frame rows, two rows as one complex
//     row, into the upper half of each frame of the chunk buffer;
//   pass 2 (k_as_col): per pair of columns kx and N - kx, DFT^- down the
//     columns, times the transfer function, DFT^+ back, in place;
//   pass 3 (k_as_row_inv): DFT^+ of every row into H (depth operand format).
// The per-frame block `asp` holds 1/lambda_t^2, a phase offset in cycles
// (dispersion) and an amplitude (gate / N^2) for each frame.
//
// The frames are real, so the spectrum S of a frame is Hermitian: only half of
// it is computed and carried.  Z_m = row m + i row (m + N/2) takes one transform
// for two rows, and columns kx and N - kx of Z hold everything of columns kx and
// N - kx of the row transforms X:
//   2 X_m[kx] = Z_m[kx] + conj Z_m[N - kx],  2 i X_{m+N/2}[kx] = Z_m[kx] - conj Z_m[N - kx]
// (rows m = j + k G, k < 8, and m + N/2 are registers k and k + 8 of the same
// thread).  S(-k) = conj S(k) and the transfer function h depends on |k| only,
// so column N - kx of the propagated spectrum needs no transform of its own:
//   DFT^+_ky[ S(-kx, ky) h ] = conj DFT^+_ky[ S(kx, ky) conj h ].
// Per pixel 2 + 4, 4 + 8 and 8 + 8 bytes instead of 2 + 8, 8 + 8 and 8 + 8, half
// of the forward transforms and half of the FP64 phases: the two passes take
// 23 + 69 us instead of 37 + 80 us per 16 frames of N = 1024.
template <int N, int SR>
__global__ __launch_bounds__(RowCfg<N>::THREADS) void k_as_row_fwd(const uint16_t* __restrict__ frames, int t0,
                                                                  const float2* __restrict__ tw,
                                                                  float2* __restrict__ inter, int rpg_) {
  using S = FFTShape<N>;
  using R = RowCfg<N>;
  constexpr int G = S::G;
  constexpr int NP = N / 2;                 // row pairs
  constexpr bool PART = R::GR > NP;         // small N: groups past the last pair repeat it and store nothing
  __shared__ float2 xbuf[R::GR][RowLds<N>::XS];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int f = blockIdx.y;
  const int rpg = SR ? SR : rpg_;
  const int m0 = (blockIdx.x * R::GR + g) * rpg;
  const uint16_t* I = frames + (size_t)(t0 + f) * N * N;
  // As in k_row_pass: the next pair loads while the current one is
  // transformed, the twiddles stay in registers, and nothing is outstanding
  // when the loop starts, so the loop waits for its prefetched pair only
  // (loaded before the previous pair's stores, which stay in flight).
  // held as 32-bit values: packing two samples per register would wait for
  // the loads (and with them the previous pair's stores) right after issue
  uint32_t nx[16], ny[16];
  auto load_pair = [&](int m) {
    if (PART && m >= NP) m = NP - 1;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      nx[k] = I[(size_t)m * N + j + k * G];
      ny[k] = I[(size_t)(m + NP) * N + j + k * G];
    }
  };
  load_pair(m0);
  const TwRegs<N> twr = load_tw_regs<N>(tw, j);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unchanged
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = make_float2((float)nx[k], (float)ny[k]);
    if (i + 1 < rpg) load_pair(m + 1);
    exchange_sync<R::WAVE>();
    fft_group_tw<N, -1, 1, R::WAVE>(v, j, xbuf[g], twr);
    float2* dst = inter + ((size_t)f * N + m) * N;
    if (!PART || m < NP) {
#pragma unroll
      for (int e = 0; e < 16; ++e) dst[j + out_offset<N>(e)] = v[e];
    }
  }
}

// The transfer-function column pass keeps 16 FP64 phase evaluations in flight
// per thread, so its tiles are narrower than the column pass's: at most 256
// threads (4 column pairs at N = 1024), which leaves room for two workgroups per
// CU (LDS: exchange buffer plus twiddle table, 48 KB at N = 1024) at up to 256
// VGPRs per thread; 8-column tiles hold one workgroup per CU.
template <int N>
struct AsColCfg {
  // (at N = 2048 twice that: tiles of 2 pairs, 16-byte row segments, ran 13 % slower per render)
  static constexpr int MAXT = N == 2048 ? 2 * SSOCT_AS_THREADS : SSOCT_AS_THREADS;
  static constexpr int C0 = ColCfg<N>::C * FFTShape<N>::G > MAXT ? MAXT / FFTShape<N>::G : ColCfg<N>::C;
  static constexpr int C = C0 < N / 2 ? C0 : N / 2;      // column pairs
  static constexpr int TILES = N / 2 / C + 1;            // per frame: pairs 0 .. N/2 - 1, and column N/2 by itself
  static constexpr int THREADS = C * FFTShape<N>::G;
};

// Register of DFT^+ input element j + G m that the forward transform's output
// register e holds (element j + out_offset(e)): m = e / L + (e % L) (16 / L)
template <int N>
__device__ __forceinline__ constexpr int as_in_slot(int e) {
  constexpr int L = FFTShape<N>::L > 1 ? FFTShape<N>::L : 1;
  return e / L + (e % L) * (16 / L);
}
static_assert(as_in_slot<1024>(5) * FFTShape<1024>::G == out_offset<1024>(5), "register permutation of N = 1024");
static_assert(as_in_slot<2048>(7) * FFTShape<2048>::G == out_offset<2048>(7), "register permutation of N = 2048");
static_assert(as_in_slot<256>(9) * FFTShape<256>::G == out_offset<256>(9), "register permutation of N = 256");

// Square root of a positive normal FP64 value (no zero, subnormal, infinity or
// NaN, so none of the range scaling of the library root): the hardware
// reciprocal-root estimate, one Goldschmidt step and two Newton corrections
// of the root, which end within an ulp.
__device__ __forceinline__ double sqrt_pos(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  double d = fma(-g, g, x);
  g = fma(d, h, g);
  d = fma(-g, g, x);
  return fma(d, h, g);
}

template <int N>
__global__ __launch_bounds__(AsColCfg<N>::THREADS) SSOCT_AS_OCC void k_as_col(float2* __restrict__ buf, int t0,
                                                                const float2* __restrict__ tw,
                                                                const double* __restrict__ asp, double inv_nd,
                                                                double z, int ntiles) {
  using S = FFTShape<N>;
  constexpr int G = S::G;
  constexpr int C = AsColCfg<N>::C;
  constexpr int NCB = AsColCfg<N>::TILES;
  // As in k_col_pass, the twiddle table goes to LDS beside the exchange
  // buffer where it fits.  With SSOCT_AS_PF the freed registers hold the
  // next tile, loaded while the current one is transformed (tiles are
  // disjoint and each belongs to one workgroup, so the prefetch never reads
  // a column that is being written in place).  Two workgroups share a
  // CU.  (Column N/2 by itself is one tile in 129 at N = 1024; carried beside
  // column 0 as one complex column and told apart through LDS it cost 1.5 %
  // more than the tile.)
  constexpr int TWN = TwPlan<N>::SIZE > 0 ? TwPlan<N>::SIZE : 1;
  constexpr bool TWL = SSOCT_COL_TWL && (S::LDS * C + TWN) * 8 <= 163840;
  constexpr bool PF = TWL && SSOCT_AS_PF;
  __shared__ float2 xbuf[S::LDS * C];
  __shared__ float2 twl[TWL ? TWN : 1];
  const int c = threadIdx.x % C, j = threadIdx.x / C;
  float2 pf[16];
  auto issue = [&](int tl) {
    const float2* cs = buf + (size_t)(tl / NCB) * N * N;
    const int kx = min((tl % NCB) * C + c, N / 2), kp = (N - kx) & (N - 1);   // the last tile repeats N/2
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      pf[k] = cs[(uint32_t)(j * N + kx) + (uint32_t)(k * G * N)];       // uniform base, 32-bit thread offsets
      pf[k + 8] = cs[(uint32_t)(j * N + kp) + (uint32_t)(k * G * N)];
    }
  };
  // tiles tile0, tile0 + tstride, ... below tend: with SSOCT_AS_XCD each XCD
  // (workgroups are dispatched round-robin over the 8) walks a contiguous run,
  // so the workgroups of one L2 hold neighbouring column blocks
  int tile0 = blockIdx.x, tstride = gridDim.x, tend = ntiles;
  if (SSOCT_AS_XCD && gridDim.x % 8 == 0) {
    const int per = (ntiles + 7) / 8, x = blockIdx.x % 8;
    tile0 = x * per + (int)blockIdx.x / 8;
    tstride = gridDim.x / 8;
    tend = min(ntiles, (x + 1) * per);
  }
  if constexpr (TWL) {
    if (PF && tile0 < tend) issue(tile0);
    for (int i = threadIdx.x; i < TwPlan<N>::SIZE; i += AsColCfg<N>::THREADS) twl[i] = tw[i];
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop is entered with no load outstanding
    __syncthreads();  // twiddles visible
  }
  const TwMem<N> twm{TWL ? static_cast<const float2*>(twl) : tw, j};
#pragma unroll 1
  for (int tile = tile0; tile < tend; tile += tstride) {
    const int f = tile / NCB, kx0 = (tile % NCB) * C + c, kx = min(kx0, N / 2);
    float2* col = buf + (size_t)f * N * N;
    if constexpr (!PF) issue(tile);
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 8; ++k) {   // 2 X of rows m and m + N/2 (the factor goes into the amplitude)
      const float2 za = pf[k], zb = pf[k + 8];
      v[k] = make_float2(za.x + zb.x, za.y - zb.y);
      v[k + 8] = make_float2(za.y + zb.y, zb.x - za.x);
    }
    if (PF && tile + tstride < tend) issue(tile + tstride);
    fft_group_tw<N, -1, C, false>(v, j, xbuf + c, twm);
    const double* fp = asp + 3 * (size_t)(t0 + f);
    const double inv_l2 = fp[0], cyc0 = fp[1], amp = 0.5 * fp[2];
    // squared spatial frequency (kx'^2 + ky'^2) / (N d)^2 from the exact integer kx'^2 + ky'^2
    // (signed indices, at most N^2 / 2)
    const int kx2 = kx * kx;                    // kx <= N/2
    const double inv_nd2 = inv_nd * inv_nd;
    const float famp = (float)amp;
    // propagating: exp(2 pi i (cyc0 - z sqrt(rad))) amp; evanescent (rad <= 0): 0
    // (exp(-i k z) for +z: the paper's fields carry exp(+i omega t), as the prefactor of Eq. 6
    // does).  The phase (up to ~1e5 cycles) is reduced to a fraction in FP64; the hardware sine
    // and cosine take the fraction in cycles (within 1.3e-7 of FP64 over one cycle on gfx950).
    // Evaluated without branches (an evanescent element takes a dummy root and is zeroed), so the
    // sixteen FP64 chains of a thread interleave.
    // The products go straight to the input order of DFT^+, which wants
    // element j + k G in register k: the forward output register e holds
    // element j + out_offset(e) = j + G m(e), m(e) = e / L + (e % L) (16 / L),
    // so the same thread already holds every element it needs and a register
    // permutation replaces an exchange (the transform's own first exchange
    // waits for the forward transform's last reads of xbuf)
    float2 w[16], wc[16];
    auto transfer = [&](int kx2, int e) {
      const int ky = j + out_offset<N>(e);
      const int sy = ky < N / 2 ? ky : ky - N;
      const double rad = inv_l2 - (double)(kx2 + sy * sy) * inv_nd2;
      const bool prop = rad > 0.0;
      double cyc = cyc0 - z * sqrt_pos(prop ? rad : 1.0);
      cyc -= rint(cyc);
      const float fr = (float)cyc;
      return make_float2(prop ? __builtin_amdgcn_cosf(fr) * famp : 0.f, prop ? __builtin_amdgcn_sinf(fr) * famp : 0.f);
    };
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float2 h = transfer(kx2, e);
      w[as_in_slot<N>(e)] = cmul(v[e], h);
      wc[as_in_slot<N>(e)] = cmulc(v[e], h);
#if SSOCT_AS_GROUP > 0
      if ((e + 1) % SSOCT_AS_GROUP == 0) __builtin_amdgcn_sched_barrier(0);
#endif
    }
    fft_group_tw<N, +1, C, false>(w, j, xbuf + c, twm);
    if (kx0 <= N / 2) {
#pragma unroll
      for (int e = 0; e < 16; ++e) col[(uint32_t)(j * N + kx) + (uint32_t)(out_offset<N>(e) * N)] = w[e];
    }
    fft_group_tw<N, +1, C, false>(wc, j, xbuf + c, twm);
    if (kx0 > 0 && kx0 < N / 2) {   // columns 0 and N/2 have no partner
#pragma unroll
      for (int e = 0; e < 16; ++e)
        col[(uint32_t)(j * N + N - kx) + (uint32_t)(out_offset<N>(e) * N)] = cconj(wc[e]);
    }
    __syncthreads();   // this tile's exchange reads are done before the next tile writes LDS
  }
}

template <int N, int FMT, int SR>
__global__ __launch_bounds__(RowCfg<N>::THREADS) void k_as_row_inv(const float2* __restrict__ inter, int t0,
                                                                  const float2* __restrict__ tw,
                                                                  void* __restrict__ H, float scale, int rpg_) {
  using S = FFTShape<N>;
  using R = RowCfg<N>;
  constexpr int G = S::G;
  __shared__ float2 xbuf[R::GR][RowLds<N>::XS];
  const int g = threadIdx.x / G, j = threadIdx.x % G;
  const int f = blockIdx.y;
  const int rpg = SR ? SR : rpg_;
  const int m0 = (blockIdx.x * R::GR + g) * rpg;
  // next row prefetched, twiddles in registers, empty entry state (k_as_row_fwd)
  float2 nx[16];
  {
    const float2* src = inter + ((size_t)f * N + m0) * N;
#pragma unroll
    for (int k = 0; k < 16; ++k) nx[k] = src[j + k * G];
  }
  const TwRegs<N> twr = load_tw_regs<N>(tw, j);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unchanged
#pragma unroll 1
  for (int i = 0; i < rpg; ++i) {
    const int m = m0 + i;
    float2 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = nx[k];
    if (i + 1 < rpg) {
      const float2* src = inter + ((size_t)f * N + m + 1) * N;
#pragma unroll
      for (int k = 0; k < 16; ++k) nx[k] = src[j + k * G];
    }
    exchange_sync<R::WAVE>();
    fft_group_tw<N, +1, 1, R::WAVE>(v, j, xbuf[g], twr);
    const long long base = ((long long)(t0 + f) * N + m) * N;
#pragma unroll
    for (int e = 0; e < 16; ++e) store_h<FMT>(H, base + j + out_offset<N>(e), v[e], scale);
  }
}

// Default persistent grid of the transfer-function column pass: one resident
// round of workgroups (its next tile is prefetched, so a second round only
// adds a tail), with the per-CU residency of the compiled kernel
template <int N>
static int as_col_default_grid_n(int cu) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(k_as_col<N>),
                                                   AsColCfg<N>::THREADS, 0) != hipSuccess || nb < 1)
    nb = 1;
  return cu * nb;
}

int as_col_default_grid(int N, int cu) {
  switch (N) {
    case 16: return as_col_default_grid_n<16>(cu);
    case 32: return as_col_default_grid_n<32>(cu);
    case 64: return as_col_default_grid_n<64>(cu);
    case 128: return as_col_default_grid_n<128>(cu);
    case 256: return as_col_default_grid_n<256>(cu);
    case 512: return as_col_default_grid_n<512>(cu);
    case 1024: return as_col_default_grid_n<1024>(cu);
    default: return as_col_default_grid_n<2048>(cu);
  }
}

template <int N>
static hipError_t as_stage_n(int F, int t0, const uint16_t* frames, const float2* tw, const double* asp,
                             double inv_nd, double z, float2* inter, void* H, int fmt, int sigma, int req_grid,
                             int cu, hipStream_t s) {
  using R = RowCfg<N>;
  using C = AsColCfg<N>;
  const int rpg = row_rpg<N>(F, cu, SSOCT_ROW_PER_CU);
  dim3 rgrid(N / (R::GR * rpg), F), rblock(R::THREADS);
  const bool full = rpg == R::RPG;
  // row pairs: half as many, so half the rows per group where that keeps the launch size (above
  // N = 64 the default chunk gives half of RPG or fewer, the run-time variant; only a chunk tuned larger gives RPG)
  constexpr int NP = N / 2;
  int rpgp = R::RPG < NP / R::GR ? R::RPG : (NP / R::GR > 1 ? NP / R::GR : 1);
  while (rpgp > 1 && (long long)(NP / (R::GR * rpgp)) * F < (long long)SSOCT_ROW_PER_CU * cu) rpgp /= 2;
  dim3 pgrid(NP > R::GR * rpgp ? NP / (R::GR * rpgp) : 1, F);
  if (rpgp == R::RPG) hipLaunchKernelGGL((k_as_row_fwd<N, R::RPG>), pgrid, rblock, 0, s, frames, t0, tw, inter, rpgp);
  else hipLaunchKernelGGL((k_as_row_fwd<N, 0>), pgrid, rblock, 0, s, frames, t0, tw, inter, rpgp);
  const int ntiles = F * C::TILES;
  hipLaunchKernelGGL((k_as_col<N>), dim3(col_grid(ntiles, req_grid)), dim3(C::THREADS), 0, s, inter, t0, tw, asp,
                     inv_nd, z, ntiles);
  const float scale = ldexpf(1.0f, -sigma);
#define SSOCT_AI(FMT)                                                                                                \
  do {                                                                                                              \
    if (full) hipLaunchKernelGGL((k_as_row_inv<N, FMT, R::RPG>), rgrid, rblock, 0, s, inter, t0, tw, H, scale, rpg); \
    else hipLaunchKernelGGL((k_as_row_inv<N, FMT, 0>), rgrid, rblock, 0, s, inter, t0, tw, H, scale, rpg);           \
  } while (0)
  if (fmt == HF_F32) SSOCT_AI(HF_F32);
  else if (fmt == HF_F16) SSOCT_AI(HF_F16);
  else SSOCT_AI(HF_BF16);
#undef SSOCT_AI
  return hipGetLastError();
}

hipError_t launch_as_stage(int N, int F, int t0, const uint16_t* frames, const float2* tw, const double* asp,
                           double inv_nd, double z, float2* inter, void* H, int fmt, int sigma, int grid,
                           int cu, hipStream_t s) {
#define CALL(n) as_stage_n<n>(F, t0, frames, tw, asp, inv_nd, z, inter, H, fmt, sigma, grid, cu, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

}  // namespace ssoct
