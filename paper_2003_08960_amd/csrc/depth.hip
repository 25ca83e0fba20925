// Depth transform (Eq. 7 with a rectangular gate over the T frames of a
// sweep) as a dense real GEMM on MFMA.
//
// The complex DFT matrix W[q][t] = exp(-2 pi i q t / T) has W_{T-q} =
// conj(W_q).  With A_q = sum_t Re(W_q[t]) h_t and B_q = sum_t Im(W_q[t]) h_t,
//     V[q]   = A_q + i B_q,     V[T-q] = A_q - i B_q,
// so one T x T real matrix whose rows are the pairs (Re W_q, Im W_q)
// (q = 1 .. T-1-T/2, plus the pair (W_0, W_{T/2})) applied to the complex
// stack viewed as reals gives the whole spectrum with 4 T^2 real flops per
// pixel instead of 8 T^2.  The adjoint (exp(+2 pi i q t / T)) swaps V[q] and
// V[T-q].
//
// A sweep not linear in k has exp(-2 pi i q kappa_t / T) instead, with kappa_t
// real.  DM_KAPPA takes a row pair per bin, 2 T real rows.  DM_KAPPA_PAIRED
// writes it about the centre c = (T - 1) / 2 of the bins, where rows pair up
// again: with p = q - c, W_p[t] = exp(-2 pi i p kappa_t / T) has
// W_{-p} = conj(W_p), and the frames carry the rest, exp(-2 pi i c kappa_t / T),
// from the Fresnel stage (a per-frame phase).  For even T p runs over
// +-1/2 .. +-(T-1)/2, for odd T over 0, +-1 .. +-(T-1)/2: T (T + 1 for odd T)
// real rows and half the products.  The MFMA rate bounds the FP32 form: a
// render of T = 256, N = 512 takes 904 us with paired rows, 1424 us without
// (FP16 split at T = 200, N = 256: 137 and 199 us).  The errors of the two against
// FP64 are alike; but they round the frames and the matrix in different places.
// In FP32 and FP16 split that moves a volume by rounding of the order of FP32's;
// in BF16 split by up to 3e-5 (a weak cut, whose whole error is 2.1e-5), and in the
// unsplit forms by more still.  A form keeps its values from one version of the
// library to the next, so these keep DM_KAPPA, although pairing would be faster
// (BF16 split at T = 256, N = 512: 824 -> 616 us when it was tried).
//
// Work split: a workgroup owns up to 256 rows (one wave per 32-row block, rows
// kept in registers for the life of the kernel) and walks 32-pixel tiles of
// the stack; each tile of KC frames x 32 pixels is staged in LDS and read by
// every wave.  Row pairs (2k, 2k+1) and the re/im columns of a pixel land in
// the same lane of the 32x32 accumulator, so the epilogue needs no exchange.
//
// While a tile is multiplied the next one is in flight to registers; how it then
// reaches LDS is chosen per form and sweep length (k_depth below).  More than
// 256 rows are split over workgroups that sit on one XCD and walk the same tiles,
// so that the stack comes from HBM once.  Idle row blocks and the zero steps past
// frame T are left out.  Bound by the stack and the volume in the 16-bit forms, by
// the MFMA rate in FP32: this kernel takes 235 us for BF16 split at T = 256, N = 512
// (4.6 TB/s), with a row pair per bin (512 rows) 392 us; FP32 at N = 512, T = 130
// 309 us (5 of 8 row blocks used; 520 with all of them), at N = 256, T = 300 398 us.
//
// Operand precisions: FP32 (v_mfma_f32_32x32x2_f32), FP16/BF16 hi only, and
// FP16/BF16 split hi*hi + hi*lo + lo*hi (v_mfma_f32_32x32x16_{f16,bf16}),
// always with FP32 accumulation.
#include "access.hpp"
#include "internal.hpp"
#include "mfma.hpp"

#ifndef SSOCT_DEPTH_NT
#define SSOCT_DEPTH_NT 0         // non-temporal loads of H and stores of the volume
#endif

namespace ssoct {

constexpr int PT = 32;  // pixels per tile

// When the next tile goes from registers to LDS: after the products of the
// current one into the same buffer (two barriers per tile), or into the other of
// two buffers before or after them (one barrier).
//
// 8 waves of 16-bit operands: each element of a tile is read by every wave, so
// the thread that loaded it packs it into MFMA operand order (8 frames of one part
// of one pixel per 16 bytes) and a wave reads a step's operands with one 16-byte
// access each; packed by every wave for itself they take 16 permutes per step and
// wave (T = 256, N = 512: 257 against 235 us; T = 200 219 against 193).  The packing
// stands between a tile's arrival and the loads after it, so the products come
// before it (mid-products or earlier: 5 .. 9 % slower).  Fewer waves leave too
// little to save: up to 4 of them pack for themselves from one buffer (T = 100 and
// 128, N = 512: 87 and 106 us, packed once 92 and 109), but for one wave of
// unsplit operands, half the LDS traffic when packed (T = 2, N = 2048: 94 and 107 us).
// FP32: one buffer, whose second barrier costs less than the tile that two
// buffers have to wait for at the start (T = 63, N = 512 and 256: 63.4 and 22.8 us
// against 71.1 and 25.9); with 256 frames per tile two buffers, filled early
// (T = 250, N = 512: 555 against 568 us; T = 200 441 against 456).
enum Hand : int { SINGLE, BEFORE, AFTER };

// Which workgroups walk which row slab: slab sl of walker w is workgroup
// (w / 8) 8 slabs + 8 sl + w % 8 where the grid allows it (workgroups are
// dispatched round-robin over the 8 XCDs: the slabs of a walker share an L2).
// A walker is one workgroup per slab, so a launch has at least `slabs` of them
// (launch_depth refuses fewer); those past the last whole walker have no tile.
__device__ __forceinline__ void depth_role(int grid, int slabs, int b, int& walkers, int& walker, int& slab) {
  if (slabs == 1) {
    walkers = grid;
    walker = b;
    slab = 0;
  } else if (grid % (8 * slabs) == 0) {
    walkers = grid / slabs;
    slab = (b / 8) % slabs;
    walker = b / (8 * slabs) * 8 + b % 8;
  } else {
    walkers = grid / slabs;
    slab = b % slabs;
    walker = b / slabs;
  }
}

template <int PREC, int KC, int WAVES, int DIR, int EPI>
__global__ __launch_bounds__(WAVES * 64) void k_depth(const uint2* __restrict__ in, const void* __restrict__ amat,
                                                      void* __restrict__ out, int T, int T_pad, int P, int slabs,
                                                      float out_scale, float gamma_scale,
                                                      double* __restrict__ loss_partials,
                                                      const float2* __restrict__ wt, int shift, int matrix) {
  using PT_ = PrecTraits<PREC>;
  constexpr int NA = PT_::F32 ? KC / 2 : (PT_::SPLIT ? KC / 2 : KC / 4);  // dwords of A per lane
  constexpr int PER_ROW = PT / 2;                                       // uint4 per tile row
  constexpr int ROWS_PER_PASS = WAVES * 64 / PER_ROW;
  // operands packed once per tile, by the thread that loaded them
  constexpr bool PACK = !PT_::F32 && (WAVES == 8 || (WAVES == 1 && !PT_::SPLIT));
  constexpr int HAND = PACK ? AFTER : (PT_::F32 && KC == 256 ? BEFORE : SINGLE);
  // prefetch registers (uint4, two pixels of one frame): rows r0 + i ROWS_PER_PASS of the tile, or (PACK)
  // the 8 frames of operand group r0
  constexpr int NLD = PACK ? 8 : (KC + ROWS_PER_PASS - 1) / ROWS_PER_PASS;
  constexpr int NV = PACK && !PT_::SPLIT ? 2 : 4;                       // uint4 of LDS per 8 frames and pixel
  constexpr int BUF = NV * (KC / 8) * PT;                               // uint4 per buffer
  static_assert(!PACK || (KC / 8) * PER_ROW <= WAVES * 64, "one operand group and pixel pair per thread");
  __shared__ uint4 bufs[HAND == SINGLE ? 1 : 2][BUF];
  __shared__ double red[WAVES];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int nch = T_pad / KC;
  const int ntp = P / PT;
  const int h = T / 2;
  const int npairs = matrix == DM_KAPPA ? T : T - h;   // DM_KAPPA: one row pair per bin
  int walkers, walker, slab;
  depth_role(gridDim.x, slabs, blockIdx.x, walkers, walker, slab);
  const int my_tiles = walker < walkers && walker < ntp ? (ntp - 1 - walker) / walkers + 1 : 0;
  const int nitems = my_tiles * nch;                                    // (tile, chunk) work items
  const int cq = threadIdx.x % PER_ROW, r0 = threadIdx.x / PER_ROW;
  const int rb = slab * WAVES + w;                                      // this wave's row block
  const bool active = rb * 16 < npairs;                                 // (a block past the last row has none)
  uint32_t a[NA];
  uint4 pf[NLD];
  double loss = 0.0;
  int a_chunk = -1;
  v16f acc_re, acc_im;

  // global loads of work item `it` (KC frames x 32 pixels) into pf, zero past T
  auto issue = [&](int it) {
    const int tile = walker + (it / nch) * walkers;
    const int ch = it % nch;
    const int p0 = tile * PT;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int r = PACK ? r0 * 8 + i : r0 + i * ROWS_PER_PASS;
      const int t = ch * KC + r;
      pf[i] = make_uint4(0u, 0u, 0u, 0u);
      if (r < KC && t < T) pf[i] = ld_once<SSOCT_DEPTH_NT>(reinterpret_cast<const uint4*>(in + (size_t)t * P + p0 + 2 * cq));
    }
  };
  // LDS: [frame][pixel] uint2; packed as [vector][group of 8 frames][pixel] uint4, the vectors being
  // re hi, im hi, re lo, im lo
  auto publish = [&](uint4* buf) {
    if constexpr (!PACK) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int r = r0 + i * ROWS_PER_PASS;
        if (r < KC) buf[r * (PT / 2) + cq] = pf[i];
      }
    } else if (r0 < KC / 8) {
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        uint32_t re[8], im[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          re[i] = o == 0 ? pf[i].x : pf[i].z;
          im[i] = o == 0 ? pf[i].y : pf[i].w;
        }
        uint4* dst = buf + r0 * PT + 2 * cq + o;
        constexpr int VS = (KC / 8) * PT;
        dst[0] = make_uint4(pack_lo(re[0], re[1]), pack_lo(re[2], re[3]), pack_lo(re[4], re[5]), pack_lo(re[6], re[7]));
        dst[VS] = make_uint4(pack_lo(im[0], im[1]), pack_lo(im[2], im[3]), pack_lo(im[4], im[5]), pack_lo(im[6], im[7]));
        if constexpr (PT_::SPLIT) {
          dst[2 * VS] = make_uint4(pack_hi(re[0], re[1]), pack_hi(re[2], re[3]), pack_hi(re[4], re[5]), pack_hi(re[6], re[7]));
          dst[3 * VS] = make_uint4(pack_hi(im[0], im[1]), pack_hi(im[2], im[3]), pack_hi(im[4], im[5]), pack_hi(im[6], im[7]));
        }
      }
    }
  };

  // this wave's matrix rows of chunk ch
  auto load_rows = [&](int ch) {
          if constexpr (PT_::F32) {
            const float* src = reinterpret_cast<const float*>(amat) + ((size_t)rb * (T_pad / 2) + ch * (KC / 2)) * 64 + l;
    #pragma unroll
            for (int s = 0; s < KC / 2; ++s) a[s] = __float_as_uint(src[(size_t)s * 64]);
          } else {
            const uint4* src = reinterpret_cast<const uint4*>(amat) + ((size_t)rb * (T_pad / 16) + ch * (KC / 16)) * 128 + l;
    #pragma unroll
            for (int s = 0; s < KC / 16; ++s) {
              const uint4 hi = src[(size_t)s * 128];
              a[(PT_::SPLIT ? 8 : 4) * s + 0] = hi.x;
              a[(PT_::SPLIT ? 8 : 4) * s + 1] = hi.y;
              a[(PT_::SPLIT ? 8 : 4) * s + 2] = hi.z;
              a[(PT_::SPLIT ? 8 : 4) * s + 3] = hi.w;
              if constexpr (PT_::SPLIT) {
                const uint4 lo = src[(size_t)s * 128 + 64];
                a[8 * s + 4] = lo.x;
                a[8 * s + 5] = lo.y;
                a[8 * s + 6] = lo.z;
                a[8 * s + 7] = lo.w;
              }
            }
          }
  };

  // the first tile and the rows it is multiplied by are in flight together; AFTER loads the rows behind
  // the first tile, as its products come to need them (N = 16, one tile per workgroup, BF16 split: T = 256
  // 15.1 us a render, 16.1 with all rows first)
  if (nitems > 0) {
    issue(0);
    if constexpr (HAND != AFTER) {
      if (active) load_rows(0);
      a_chunk = 0;
    }
    if constexpr (HAND != SINGLE) {
      publish(bufs[0]);
      if (nitems > 1) issue(1);
    }
  }
  if constexpr (HAND == AFTER) __syncthreads();
  for (int it = 0; it < nitems; ++it) {
    const int tile = walker + (it / nch) * walkers;
    const int ch = it % nch;
    const int p0 = tile * PT;
    const uint4* buf = bufs[HAND == SINGLE ? 0 : it & 1];
    if (ch == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc_re[i] = 0.f;
        acc_im[i] = 0.f;
      }
    }
    if (a_chunk != ch && active) {   // several chunks: the rows of each in turn
      load_rows(ch);
      a_chunk = ch;
    }
    if constexpr (HAND == SINGLE) {
      __syncthreads();               // the previous tile's reads are done
      publish(bufs[0]);
      __syncthreads();
      if (it + 1 < nitems) issue(it + 1);
    } else if constexpr (HAND == BEFORE) {
      __syncthreads();               // this tile is there, and the previous one's reads are done
      if (it + 1 < nitems) publish(bufs[(it + 1) & 1]);
      if (it + 2 < nitems) issue(it + 2);
    }
    // ---- MFMA over the chunk; steps past frame T hold zeros and are left out (groups of DS steps)
    const int kt = T - ch * KC;
    if (active) {
      if constexpr (PT_::F32) {
        // the next group's operands are read while this group multiplies (a group is a block of its own)
        constexpr int DS = 4, NG = KC / (2 * DS);
        const uint2* bl = reinterpret_cast<const uint2*>(buf) + l;   // lanes 0..31: even frames, 32..63: odd ones
        uint2 b[2][DS];
#pragma unroll
        for (int i = 0; i < DS; ++i) b[0][i] = bl[2 * i * PT];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          if (g * 2 * DS < kt) {
            if (g + 1 < NG) {
#pragma unroll
              for (int i = 0; i < DS; ++i) b[(g + 1) & 1][i] = bl[2 * ((g + 1) * DS + i) * PT];
            }
#pragma unroll
            for (int i = 0; i < DS; ++i) {
              const float av = __uint_as_float(a[g * DS + i]);
              acc_re = __builtin_amdgcn_mfma_f32_32x32x2f32(av, __uint_as_float(b[g & 1][i].x), acc_re, 0, 0, 0);
              acc_im = __builtin_amdgcn_mfma_f32_32x32x2f32(av, __uint_as_float(b[g & 1][i].y), acc_im, 0, 0, 0);
            }
          }
        }
      } else {
        constexpr int VS = (KC / 8) * PT;
        constexpr int DS = PACK && KC > 64 ? 4 : KC / 16;
#pragma unroll
        for (int g = 0; g < KC / (16 * DS); ++g) {
          if (g * 16 * DS < kt) {
#pragma unroll
            for (int s = g * DS; s < (g + 1) * DS; ++s) {
              // lanes 0..31: frames 16 s + 0..7, 32..63: + 8..15
              uint4 re_hi, im_hi, re_lo, im_lo;
              if constexpr (PACK) {
                const uint4* e = buf + (2 * s) * PT + l;
                re_hi = e[0], im_hi = e[VS];
                if constexpr (PT_::SPLIT) re_lo = e[2 * VS], im_lo = e[3 * VS];
              } else {
                uint2 e[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                  e[i] = reinterpret_cast<const uint2*>(buf)[(16 * s + 8 * (l >> 5) + i) * PT + (l & 31)];
                re_hi = make_uint4(pack_lo(e[0].x, e[1].x), pack_lo(e[2].x, e[3].x), pack_lo(e[4].x, e[5].x), pack_lo(e[6].x, e[7].x));
                im_hi = make_uint4(pack_lo(e[0].y, e[1].y), pack_lo(e[2].y, e[3].y), pack_lo(e[4].y, e[5].y), pack_lo(e[6].y, e[7].y));
                if constexpr (PT_::SPLIT) {
                  re_lo = make_uint4(pack_hi(e[0].x, e[1].x), pack_hi(e[2].x, e[3].x), pack_hi(e[4].x, e[5].x), pack_hi(e[6].x, e[7].x));
                  im_lo = make_uint4(pack_hi(e[0].y, e[1].y), pack_hi(e[2].y, e[3].y), pack_hi(e[4].y, e[5].y), pack_hi(e[6].y, e[7].y));
                }
              }
              const int ai = (PT_::SPLIT ? 8 : 4) * s;
              const uint4 ahi = make_uint4(a[ai], a[ai + 1], a[ai + 2], a[ai + 3]);
              if constexpr (PT_::SPLIT) {
                const uint4 alo = make_uint4(a[ai + 4], a[ai + 5], a[ai + 6], a[ai + 7]);
                acc_re = mfma_x16<PT_::BF>(alo, re_hi, acc_re);
                acc_im = mfma_x16<PT_::BF>(alo, im_hi, acc_im);
                acc_re = mfma_x16<PT_::BF>(ahi, re_lo, acc_re);
                acc_im = mfma_x16<PT_::BF>(ahi, im_lo, acc_im);
              }
              acc_re = mfma_x16<PT_::BF>(ahi, re_hi, acc_re);
              acc_im = mfma_x16<PT_::BF>(ahi, im_hi, acc_im);
            }
          }
        }
      }
    }
    if constexpr (HAND == AFTER) {   // the next tile's loads are older than any store below
      if (it + 1 < nitems) publish(bufs[(it + 1) & 1]);
      if (it + 2 < nitems) issue(it + 2);
      __syncthreads();
    }
    if (ch != nch - 1 || !active) continue;
    // ---- epilogue: lane holds rows 8 (r/4) + 4 (l/32) + r%4 of its block, column l%32
    const int p = p0 + (l & 31);
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const int row = rb * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
      const int k = row >> 1;
      if (k >= npairs) continue;
      const float Ar = acc_re[r] * out_scale, Ai = acc_im[r] * out_scale;
      const float Br = acc_re[r + 1] * out_scale, Bi = acc_im[r + 1] * out_scale;
      float2 v1, v2;
      int q1, q2;
      if (matrix == DM_KAPPA) {   // V[k] = A + i B
        q1 = k; v1 = make_float2(Ar - Bi, Ai + Br);
        q2 = -1; v2 = v1;
      } else if (matrix == DM_KAPPA_PAIRED) {   // bins c + p and c - p, c = (T - 1) / 2, p = k + 1/2 (even T) or k
        q1 = h + k; v1 = make_float2(Ar - Bi, Ai + Br);
        q2 = T % 2 == 0 ? h - 1 - k : (k > 0 ? h - k : -1); v2 = make_float2(Ar + Bi, Ai - Br);
      } else if (k == 0) {
        q1 = 0; v1 = make_float2(Ar, Ai);
        q2 = (T % 2 == 0) ? h : -1; v2 = make_float2(Br, Bi);
      } else {
        const float2 vq = make_float2(Ar - Bi, Ai + Br);
        const float2 vm = make_float2(Ar + Bi, Ai - Br);
        q1 = k; q2 = T - k;
        v1 = DIR > 0 ? vq : vm;
        v2 = DIR > 0 ? vm : vq;
      }
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int q = o == 0 ? q1 : q2;
        if (q < 0) continue;
        float2 V = o == 0 ? v1 : v2;
        const size_t idx = (size_t)q * P + p;
        if constexpr (EPI == EPI_STORE) {
          // window starting `shift` frames into the ring: bin q gains exp(+2 pi i q shift / T)
          if (DIR > 0 && shift != 0) {
            const float2 w = wt[(q * shift) % T];   // V conj(w)
            V = make_float2(V.x * w.x + V.y * w.y, V.y * w.x - V.x * w.y);
          }
          st_once<SSOCT_DEPTH_NT>(reinterpret_cast<float2*>(out) + idx, V);
        } else if constexpr (EPI == EPI_ABS) {
          st_once<SSOCT_DEPTH_NT>(reinterpret_cast<float*>(out) + idx, sqrtf(V.x * V.x + V.y * V.y));
        } else {
          const double a2 = (double)V.x * V.x + (double)V.y * V.y;
          loss += a2 * a2;
          const float sx = V.x * gamma_scale, sy = V.y * gamma_scale;
          const float m2 = 4.0f * (sx * sx + sy * sy);
          reinterpret_cast<float2*>(out)[idx] = make_float2(m2 * sx, m2 * sy);
        }
      }
    }
  }
  if constexpr (EPI == EPI_GAMMA) {
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
    if (l == 0) red[w] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int i = 0; i < WAVES; ++i) s += red[i];
      loss_partials[blockIdx.x] = s;
    }
  }
}

template <int PREC, int KC, int WAVES, int DIR, int EPI>
static hipError_t depth_go(int grid, hipStream_t s, const void* in, const void* amat, void* out, int T, int T_pad,
                           int P, int slabs, float out_scale, float gamma_scale, double* partials, const float2* wt,
                           int shift, int matrix) {
  hipLaunchKernelGGL((k_depth<PREC, KC, WAVES, DIR, EPI>), dim3(grid), dim3(WAVES * 64), 0, s,
                     reinterpret_cast<const uint2*>(in), amat, out, T, T_pad, P, slabs, out_scale, gamma_scale,
                     partials, wt, shift, matrix);
  return hipGetLastError();
}

template <int PREC, int KC, int WAVES>
static hipError_t depth_dir_epi(int dir, int epi, int grid, hipStream_t s, const void* in, const void* amat,
                                void* out, int T, int T_pad, int P, int slabs, float os, float gs, double* part, const float2* wt, int shift, int matrix) {
  if (dir > 0) {
    if (epi == EPI_STORE) return depth_go<PREC, KC, WAVES, +1, EPI_STORE>(grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    if (epi == EPI_ABS) return depth_go<PREC, KC, WAVES, +1, EPI_ABS>(grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    if constexpr (PREC == DP_F32)
      return depth_go<PREC, KC, WAVES, +1, EPI_GAMMA>(grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    return hipErrorInvalidValue;
  }
  if constexpr (PREC == DP_F32) {
    if (epi == EPI_STORE) return depth_go<PREC, KC, WAVES, -1, EPI_STORE>(grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
  }
  return hipErrorInvalidValue;
}

// KC and waves as depth_layout gives them (32 waves >= KC: a row block and a
// thread per operand group), and half the KC of those
template <int PREC, int KC>
static hipError_t depth_waves(int waves, int dir, int epi, int grid, hipStream_t s, const void* in, const void* amat,
                              void* out, int T, int T_pad, int P, int slabs, float os, float gs, double* part, const float2* wt, int shift, int matrix) {
#define SSOCT_DW(W)                                                                                                  \
  if constexpr (32 * W >= KC && 32 * W <= 4 * KC)                                                                    \
    if (waves == W)                                                                                                  \
      return depth_dir_epi<PREC, KC, W>(dir, epi, grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, \
                                        matrix);
  SSOCT_DW(1)
  SSOCT_DW(2)
  SSOCT_DW(4)
  SSOCT_DW(8)
#undef SSOCT_DW
  return hipErrorInvalidValue;
}

template <int PREC>
static hipError_t depth_kc(int KC, int waves, int dir, int epi, int grid, hipStream_t s, const void* in,
                           const void* amat, void* out, int T, int T_pad, int P, int slabs, float os, float gs,
                           double* part, const float2* wt, int shift, int matrix) {
  switch (KC) {
    case 32: return depth_waves<PREC, 32>(waves, dir, epi, grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    case 64: return depth_waves<PREC, 64>(waves, dir, epi, grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    case 128: return depth_waves<PREC, 128>(waves, dir, epi, grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    case 256: return depth_waves<PREC, 256>(waves, dir, epi, grid, s, in, amat, out, T, T_pad, P, slabs, os, gs, part, wt, shift, matrix);
    default: return hipErrorInvalidValue;
  }
}

int depth_grid(int T, int P, int cu_count, int matrix) {
  DepthLayout L = depth_layout(T, matrix);
  const int ntiles = (P / PT) * L.slabs;
  int per_cu = 8 / L.waves;          // waves per CU target ~8
  if (per_cu < 1) per_cu = 1;
  const int g = cu_count * per_cu;
  return ntiles < g ? ntiles : g;
}

hipError_t launch_depth(int T, int P, int prec, int dir, int epi, const void* in, const void* amat, void* out,
                        int sigma, int gamma_exp, double* partials, int grid, hipStream_t s, const float2* wt,
                        int shift, int matrix, int kc) {
  if (shift != 0 && !wt) return hipErrorInvalidValue;
  if (matrix != DM_DFT && (dir < 0 || epi == EPI_GAMMA || shift != 0)) return hipErrorInvalidValue;   // forward only
  DepthLayout L = depth_layout(T, matrix);
  // a smaller K chunk that divides the layout's keeps T_pad and the matrix layout (the K sum runs
  // through the same products in the same order, chunk after chunk)
  if (kc != 0) {
    if (kc < 32 || kc > L.KC || L.KC % kc != 0) return hipErrorInvalidValue;
    L.KC = kc;
  }
  if (grid < L.slabs) return hipErrorInvalidValue;   // a slab without a workgroup would not be computed
  const float os = ldexpf(1.0f, sigma);
  const float gs = ldexpf(1.0f, -gamma_exp);
  switch (prec) {
    case DP_F32: return depth_kc<DP_F32>(L.KC, L.waves, dir, epi, grid, s, in, amat, out, T, L.T_pad, P, L.slabs, os, gs, partials, wt, shift, matrix);
    case DP_F16: return depth_kc<DP_F16>(L.KC, L.waves, dir, epi, grid, s, in, amat, out, T, L.T_pad, P, L.slabs, os, gs, partials, wt, shift, matrix);
    case DP_BF16: return depth_kc<DP_BF16>(L.KC, L.waves, dir, epi, grid, s, in, amat, out, T, L.T_pad, P, L.slabs, os, gs, partials, wt, shift, matrix);
    case DP_F16_SPLIT: return depth_kc<DP_F16_SPLIT>(L.KC, L.waves, dir, epi, grid, s, in, amat, out, T, L.T_pad, P, L.slabs, os, gs, partials, wt, shift, matrix);
    case DP_BF16_SPLIT: return depth_kc<DP_BF16_SPLIT>(L.KC, L.waves, dir, epi, grid, s, in, amat, out, T, L.T_pad, P, L.slabs, os, gs, partials, wt, shift, matrix);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ssoct
