// Column passes of the Fresnel stage: the column DFT, which writes the hologram
// stack H[t][pixel] in the operand format of the depth transform (or the volume,
// depth-first order), and its adjoint (DIR = -1) for the gradient.  A column
// workgroup loads its next column tile while it transforms the current one.
#include "stage.hpp"

namespace ssoct {

#ifndef SSOCT_COL_NT_LD
#define SSOCT_COL_NT_LD 1        // column pass: non-temporal loads of the intermediate
#endif
#ifndef SSOCT_ADJ_NT
#define SSOCT_ADJ_NT 0           // adjoint column pass: non-temporal stores of the intermediate the
                                 // adjoint row pass reads back (a chunk sized to stay in MALL)
#endif

// ------------------------------------------------------------------ column pass (both directions)
// Tiles are (frame f, block of C columns) over the F frames of the launch,
// walked persistently.  Frames f < nA read src + f N^2 and write frame
// f fstride of dst; frames f >= nA read src2 + (f - nA) N^2 and write frame
// (f - nA) fstride2 of dst2, the first of them at frame first2 instead (two runs
// of frames in one launch).
// DIR = +1 writes H in format FMT (and the Eq. 6 output phase when EQ6);
// DIR = -1 writes complex64.  PL is the radix order of the transforms.
template <int N, int DIR, int FMT, bool EQ6, int CT = ColCfg<N>::C, int PL = 0>
__global__ __launch_bounds__(CT * FFTShape<N>::G) void k_col_pass(const float2* __restrict__ src,
                                                                  const float2* __restrict__ tw,
                                                                  const float2* __restrict__ outfac,
                                                                  void* __restrict__ dst, float scale, int ntiles,
                                                                  int fstride, const float2* __restrict__ src2,
                                                                  void* __restrict__ dst2, int nA, int fstride2,
                                                                  int first2) {
  using S = FFTShape<N>;
  constexpr int G = S::G;
  constexpr int C = CT;
  constexpr int W = ColWide<N, CT>::W;   // columns per thread
  constexpr int NCB = N / (C * W);       // column blocks per frame
  // The twiddle table goes to LDS where the exchange buffer leaves room for
  // it (at N = 2048, where an 8-column exchange buffer takes 139 of the 160 KB,
  // without its repeated entries).  That frees the registers the twiddles would hold for a
  // prefetch of the next tile, which then loads while the current one is
  // transformed: one 1024-thread workgroup fills a CU, so without it the
  // CU's memory and ALUs take turns.
  using LT = ColLdsT<N, CT, PL>;
  constexpr bool TWL = LT::TWL;
  constexpr bool PF = LT::PF;
  __shared__ float2 xbuf[LT::XB];
  __shared__ float2 twl[TWL ? LT::TWN : 1];
  const int c = threadIdx.x % C, j = threadIdx.x / C;
  float2 pf[W][16];
  auto issue = [&](int tile) {
    const int f = tile / NCB;
    // uniform base and 32-bit thread offsets
    const float2* s = (f < nA ? src + (size_t)f * N * N : src2 + (size_t)(f - nA) * N * N) + (tile % NCB) * (C * W);
    const uint32_t o = (uint32_t)(j * N + c * W);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if constexpr (W == 2) {
        const uint4 q = ld_once<SSOCT_COL_NT_LD>(reinterpret_cast<const uint4*>(s + (o + (uint32_t)(k * G * N))));
        pf[0][k] = make_float2(__uint_as_float(q.x), __uint_as_float(q.y));
        pf[W - 1][k] = make_float2(__uint_as_float(q.z), __uint_as_float(q.w));
      } else {
        pf[0][k] = ld_once<SSOCT_COL_NT_LD>(s + (o + (uint32_t)(k * G * N)));
      }
    }
  };
  int tile = blockIdx.x;
  if (PF && tile < ntiles) issue(tile);
  if constexpr (TWL) {
    if constexpr (LT::SMALL) {
      for (int i = threadIdx.x; i < TwSmall<N>::SIZE; i += (CT * G)) twl[i] = tw[TwSmall<N>::source(i)];
    } else {
      for (int i = threadIdx.x; i < TwPlan<N, PL>::SIZE; i += (CT * G)) twl[i] = tw[i];
    }
    // the first tile has landed; the loop is entered with no load
    // outstanding, so waiting for a prefetched tile inside it leaves the
    // previous tile's stores in flight
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unchanged
    __syncthreads();  // twiddles visible
  }
#pragma unroll 1
  for (; tile < ntiles; tile += gridDim.x) {
    float2 v[W][16];
    if constexpr (!PF) issue(tile);
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int k = 0; k < 16; ++k) v[w][k] = pf[w][k];
    if (PF && tile + (int)gridDim.x < ntiles) issue(tile + gridDim.x);
    const int f = tile / NCB;
    if constexpr (W > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int w = 0; w < W; ++w) {   // one exchange buffer, one column after the other
      if constexpr (TWL && LT::SMALL) fft_group_tw<N, DIR, C, false>(v[w], j, xbuf + c, TwSmall<N>{twl, j});
      else if constexpr (TWL) fft_group_tw<N, DIR, C, false>(v[w], j, xbuf + c, TwMem<N, PL>{twl, j});
      else fft_group_tw<N, DIR, C, false>(v[w], j, xbuf + c, TwMem<N, PL>{tw, j});
      if constexpr (W > 1) __builtin_amdgcn_sched_barrier(0);   // interleaved, the two would not fit the registers
    }
    const long long fo = (f < nA ? (long long)f * fstride
                                 : (f == nA ? (long long)first2 : (long long)(f - nA) * fstride2)) * N * N;
    using El = typename HElem<FMT>::T;
    El* d = reinterpret_cast<El*>(f < nA ? dst : dst2) + fo + (tile % NCB) * (C * W);
    const uint32_t o = (uint32_t)(j * N + c * W);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int u = j + out_offset<N, PL>(e);
      float2 val[W];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        val[w] = v[w][e];
        if constexpr (EQ6) val[w] = cmul(val[w], outfac[u]);
      }
      store_h_cols<FMT, W, (DIR > 0 ? SSOCT_COL_NT : SSOCT_ADJ_NT)>(d, o + (uint32_t)(out_offset<N, PL>(e) * N), val, scale);
    }
  }
}

template <int N, int CT>
static int col_default_grid_nt(int cu) {
  // with the tile prefetch: one resident round of workgroups, each walking
  // its tiles; without it, two rounds
  constexpr int per_lds = 163840 / ColLdsT<N, CT>::BYTES;
  constexpr int per_thr = 2048 / (CT * FFTShape<N>::G);   // at most 32 waves per CU
  constexpr int per_cu = per_lds < per_thr ? per_lds : per_thr;
  return ColLdsT<N, CT>::PF ? cu * (per_cu > 0 ? per_cu : 1) : 512;
}

template <int N>
static int col_default_grid_n(int cu, int ct) {
  using K = ColTiles<N>;
  if (ct == K::C2 && K::ALT) return col_default_grid_nt<N, K::C2>(cu);
  if (ct == K::C4 && K::ALT) return col_default_grid_nt<N, K::C4>(cu);
  return col_default_grid_nt<N, K::C>(cu);
}

int col_default_grid(int N, int cu, int ct) {
  switch (N) {
    case 16: return col_default_grid_n<16>(cu, ct);
    case 32: return col_default_grid_n<32>(cu, ct);
    case 64: return col_default_grid_n<64>(cu, ct);
    case 128: return col_default_grid_n<128>(cu, ct);
    case 256: return col_default_grid_n<256>(cu, ct);
    case 512: return col_default_grid_n<512>(cu, ct);
    case 1024: return col_default_grid_n<1024>(cu, ct);
    default: return col_default_grid_n<2048>(cu, ct);
  }
}

template <int N>
static void col_tiles_n(int* out) {
  using K = ColTiles<N>;
  out[0] = K::C;
  out[1] = K::ALT ? K::C2 : 0;
  out[2] = K::ALT ? K::C4 : 0;
}

void col_tiles(int N, int* out) {
  switch (N) {
    case 16: return col_tiles_n<16>(out);
    case 32: return col_tiles_n<32>(out);
    case 64: return col_tiles_n<64>(out);
    case 128: return col_tiles_n<128>(out);
    case 256: return col_tiles_n<256>(out);
    case 512: return col_tiles_n<512>(out);
    case 1024: return col_tiles_n<1024>(out);
    default: return col_tiles_n<2048>(out);
  }
}

// forward column pass of tile width CT and radix order PL (with the Eq. 6
// output phase when outfac is given)
template <int N, int CT, int PL>
static hipError_t col_pass_ntp(int F, const float2* inter, const float2* tw, const float2* outfac, void* dst, int fmt,
                               float scale, int req_grid, int fstride, hipStream_t s, int F2,
                               const float2* inter2, void* dst2, int fstride2, int first2) {
  const int ntiles = (F + F2) * (N / (CT * ColWide<N, CT>::W));
  dim3 grid(col_grid(ntiles, req_grid)), block(CT * FFTShape<N>::G);
#define SSOCT_COL(FMT, E)                                                                                            \
  hipLaunchKernelGGL((k_col_pass<N, +1, FMT, E, CT, PL>), grid, block, 0, s, inter, tw, outfac, dst, scale, ntiles, \
                     fstride, inter2, dst2, F, fstride2, first2)
  if (fmt == HF_F32) { if (outfac) SSOCT_COL(HF_F32, true); else SSOCT_COL(HF_F32, false); }
  else if (fmt == HF_F16) { if (outfac) SSOCT_COL(HF_F16, true); else SSOCT_COL(HF_F16, false); }
  else if (fmt == HF_ABS) { if (outfac) SSOCT_COL(HF_ABS, true); else SSOCT_COL(HF_ABS, false); }
  else { if (outfac) SSOCT_COL(HF_BF16, true); else SSOCT_COL(HF_BF16, false); }
#undef SSOCT_COL
  return hipGetLastError();
}

// the same for a runtime radix order (sizes that are a power of 16 have one)
template <int N, int CT>
static hipError_t col_pass_nt(int F, const float2* inter, const float2* tw, const float2* outfac, void* dst, int fmt,
                              float scale, int req_grid, int fstride, hipStream_t s, int F2 = 0,
                              const float2* inter2 = nullptr, void* dst2 = nullptr, int fstride2 = 0,
                              int radix = 0, int first2 = 0) {
  if constexpr (FFTShape<N>::L > 1) {
    if (radix == 1)
      return col_pass_ntp<N, CT, 1>(F, inter, tw, outfac, dst, fmt, scale, req_grid, fstride, s, F2, inter2, dst2,
                                    fstride2, first2);
  }
  if (radix != 0) return hipErrorInvalidValue;
  return col_pass_ntp<N, CT, 0>(F, inter, tw, outfac, dst, fmt, scale, req_grid, fstride, s, F2, inter2, dst2,
                                fstride2, first2);
}

// 16-byte accesses of two columns per thread need 16-byte aligned buffers (the
// offsets are multiples of 16 bytes); others, e.g. a volume at an odd complex64
// of an allocation, take the narrower tile of one column per thread
static bool cols_aligned(const void* a, const void* b, const void* c, const void* d) {
  return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c) |
           reinterpret_cast<uintptr_t>(d)) & 15) == 0;
}

// ctile: column tile width (the default ColCfg<N>::C, or one of the narrower
// ColTiles alternatives)
template <int N>
static hipError_t col_pass_n(int F, int t0, const float2* inter, const float2* tw, const float2* outfac, void* H,
                             int fmt, int sigma, int req_grid, int ctile, int radix, hipStream_t s) {
  using K = ColTiles<N>;
  const float scale = ldexpf(1.0f, -sigma);
  char* dst = reinterpret_cast<char*>(H) + (size_t)t0 * N * N * 8;
#define SSOCT_COLN(CT) col_pass_nt<N, CT>(F, inter, tw, outfac, dst, fmt, scale, req_grid, 1, s, 0, nullptr, nullptr, 0, radix)
  if (ColWide<N, K::C>::W > 1 && !ctile && !cols_aligned(inter, dst, nullptr, nullptr)) ctile = K::C2;
  if (K::ALT && ctile == K::C2) return SSOCT_COLN(K::C2);
  if (K::ALT && ctile == K::C4) return SSOCT_COLN(K::C4);
  return SSOCT_COLN(K::C);
#undef SSOCT_COLN
}

template <int N, int CT>
static hipError_t col_pass_adj_nt(int F, const float2* src, const float2* tw, float2* inter, int req_grid,
                                  hipStream_t s) {
  const int ntiles = F * (N / (CT * ColWide<N, CT>::W));
  dim3 grid(col_grid(ntiles, req_grid)), block(CT * FFTShape<N>::G);
  hipLaunchKernelGGL((k_col_pass<N, -1, HF_F32, false, CT>), grid, block, 0, s, src, tw, (const float2*)nullptr,
                     (void*)inter, 1.0f, ntiles, 1, (const float2*)nullptr, (void*)nullptr, F, 0, 0);
  return hipGetLastError();
}

template <int N>
static hipError_t col_pass_adj_n(int F, int t0, const float2* B, const float2* tw, float2* inter, int req_grid,
                                 hipStream_t s) {
  using K = ColTiles<N>;
  const float2* src = B + (size_t)t0 * N * N;
  if constexpr (ColWide<N, K::C>::W > 1) {
    if (!cols_aligned(src, inter, nullptr, nullptr)) return col_pass_adj_nt<N, K::C2>(F, src, tw, inter, req_grid, s);
  }
  return col_pass_adj_nt<N, K::C>(F, src, tw, inter, req_grid, s);
}

template <int N>
static hipError_t col_pass_v_n(int F, const float2* inter, const float2* tw, const float2* outfac, void* V, int fmt,
                               int fstride, int req_grid, int ctile, hipStream_t s, int F2, const float2* inter2,
                               void* V2, int fstride2, int radix, int first2) {
  using K = ColTiles<N>;
#define SSOCT_COLV(CT) \
  col_pass_nt<N, CT>(F, inter, tw, outfac, V, fmt, 1.0f, req_grid, fstride, s, F2, inter2, V2, fstride2, radix, first2)
  if (ColWide<N, K::C>::W > 1 && !ctile && !cols_aligned(inter, V, inter2, V2)) ctile = K::C2;
  if (K::ALT && ctile == K::C2) return SSOCT_COLV(K::C2);
  if (K::ALT && ctile == K::C4) return SSOCT_COLV(K::C4);
  return SSOCT_COLV(K::C);
#undef SSOCT_COLV
}

hipError_t launch_col_pass(int N, int F, int t0, const float2* inter, const float2* tw, const float2* outfac, void* H,
                           int fmt, int sigma, int grid, hipStream_t s, int ctile, int radix) {
#define CALL(n) col_pass_n<n>(F, t0, inter, tw, outfac, H, fmt, sigma, grid, ctile, radix, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

hipError_t launch_col_pass_adj(int N, int F, int t0, const float2* B, const float2* tw, float2* inter, int grid,
                               hipStream_t s) {
#define CALL(n) col_pass_adj_n<n>(F, t0, B, tw, inter, grid, s)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

hipError_t launch_col_pass_v(int N, int F, const float2* inter, const float2* tw, const float2* outfac, void* V,
                             int fmt, int fstride, int grid, int ctile, hipStream_t s, int F2, const float2* inter2,
                             void* V2, int fstride2, int radix, int first2) {
  if (fmt != HF_F32 && fmt != HF_ABS) return hipErrorInvalidValue;
  if (F2 > 0 && !(inter2 && V2)) return hipErrorInvalidValue;
#define CALL(n) col_pass_v_n<n>(F, inter, tw, outfac, V, fmt, fstride, grid, ctile, s, F2, inter2, V2, fstride2, radix, first2)
  SSOCT_DISPATCH_N(N, CALL)
#undef CALL
}

}  // namespace ssoct
