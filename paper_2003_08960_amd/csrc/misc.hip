// Envelope cuts (text after Eq. 7: three orthogonal cuts of the magnitude of
// the rendered volume at user-selected positions) and the final FP64
// reduction of the sharpness gradient.
#include "internal.hpp"

namespace ssoct {

// One thread per output value: N*N (xy) + T*N (xz) + T*N (yz).
__global__ void k_cuts(int T, int N, const float2* __restrict__ vol, int x0, int y0, int q0, int power,
                       float* __restrict__ cut_xy, float* __restrict__ cut_xz, float* __restrict__ cut_yz) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t nxy = (size_t)N * N, nz = (size_t)T * N;
  size_t src;
  float* dst;
  if (i < nxy) {
    src = (size_t)q0 * nxy + i;
    dst = cut_xy + i;
  } else if (i < nxy + nz) {
    const size_t k = i - nxy, q = k / N, v = k % N;
    src = q * nxy + (size_t)y0 * N + v;
    dst = cut_xz + k;
  } else if (i < nxy + 2 * nz) {
    const size_t k = i - nxy - nz, q = k / N, u = k % N;
    src = q * nxy + u * N + x0;
    dst = cut_yz + k;
  } else {
    return;
  }
  const float2 v = vol[src];
  const float m2 = v.x * v.x + v.y * v.y;
  *dst = power ? m2 : sqrtf(m2);
}

hipError_t launch_cuts(int T, int N, const float2* vol, int x0, int y0, int q0, int power, float* cut_xy,
                       float* cut_xz, float* cut_yz, hipStream_t s) {
  const size_t n = (size_t)N * N + 2 * (size_t)T * N;
  const int block = 256;
  hipLaunchKernelGGL(k_cuts, dim3((unsigned)((n + block - 1) / block)), dim3(block), 0, s, T, N, vol, x0, y0, q0,
                     power, cut_xy, cut_xz, cut_yz);
  return hipGetLastError();
}

// Reduction of the gradient in two launches.  mono_partials[t][nblk][15] are
// per-block moments M_ab = sum Im(conj(g) z) x^a y^b; zmat[j][k] expands
// Zernike j in the monomials.  Gradients (chain of the sharpness loss):
//   dL/dphi_t = -M_00(t),  dL/dz = -sum_t (alpha_t / z) (N^2 / 2) (M_20 + M_02)(t),
//   dL/dc_j   = -sum_t sum_k zmat[j][k] M_k(t),   all times grad_scale.
// Workgroup t < T of the first kernel sums the moments of frame t, the last
// GRAD_LOSS_BLOCKS sum slices of the loss partials; the second kernel, one
// workgroup, sums those.  (One workgroup for everything took 16 us at T = 128,
// N = 512, 3 % of a gradient, waiting for one CU's loads.)  Every sum runs in
// a fixed order, so the result does not depend on timing.
constexpr int GF_GROUPS = 16;                        // moment sums: 16 groups of N_MONO threads
constexpr int GF_THREADS = 256;
static_assert(GF_GROUPS * N_MONO <= GF_THREADS, "one thread per group and moment");

__global__ __launch_bounds__(GF_THREADS) void k_grad_frames(int T, int nblk, const double* __restrict__ mono_partials,
                                                            const double* __restrict__ loss_partials, int n_loss,
                                                            double grad_scale, double* __restrict__ sums,
                                                            double* __restrict__ out) {
  __shared__ double red[GF_THREADS];
  const int tid = threadIdx.x;
  double a = 0.0;
  if ((int)blockIdx.x < T) {
    const int t = blockIdx.x, g = tid / N_MONO, k = tid % N_MONO;
    if (g < GF_GROUPS) {
      const double* src = mono_partials + (size_t)t * nblk * N_MONO + k;
#pragma unroll 4
      for (int b = g; b < nblk; b += GF_GROUPS) a += src[(size_t)b * N_MONO];
    }
    red[tid] = a;
    __syncthreads();
    if (tid < N_MONO) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < GF_GROUPS; ++i) s += red[i * N_MONO + tid];
      sums[(size_t)t * N_MONO + tid] = s;
      if (tid == 0) out[1 + 1 + 15 + t] = -grad_scale * s;
    }
  } else {
    const int slice = blockIdx.x - T;
    const int per = (n_loss + GRAD_LOSS_BLOCKS - 1) / GRAD_LOSS_BLOCKS;
    const int end = min(n_loss, (slice + 1) * per);
#pragma unroll 4
    for (int i = slice * per + tid; i < end; i += GF_THREADS) a += loss_partials[i];
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (tid % 64 == 0) red[tid / 64] = a;
    __syncthreads();
    if (tid == 0) sums[(size_t)T * N_MONO + slice] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

__global__ __launch_bounds__(GF_THREADS) void k_grad_finish(int T, int N, const double* __restrict__ sums,
                                                            const double* __restrict__ alpha_over_z,
                                                            const double* __restrict__ zmat, double grad_scale,
                                                            int has_loss, double* __restrict__ out) {
  __shared__ double red[2][GF_THREADS];
  __shared__ double M[N_MONO], W[N_MONO];
  __shared__ double zs[15 * N_MONO];
  const int tid = threadIdx.x, g = tid / N_MONO, k = tid % N_MONO;
  if (tid < 15 * N_MONO) zs[tid] = zmat[tid];   // in flight while the sums are added
  double a = 0.0, w = 0.0;
  if (g < GF_GROUPS) {
#pragma unroll 4
    for (int t = g; t < T; t += GF_GROUPS) {
      const double m = sums[(size_t)t * N_MONO + k];
      a += m;
      w += alpha_over_z[t] * m;
    }
  }
  red[0][tid] = a;
  red[1][tid] = w;
  __syncthreads();
  if (tid < N_MONO) {
    double s = 0.0, v = 0.0;
#pragma unroll
    for (int i = 0; i < GF_GROUPS; ++i) {
      s += red[0][i * N_MONO + tid];
      v += red[1][i * N_MONO + tid];
    }
    M[tid] = s;
    W[tid] = v;
  }
  __syncthreads();
  if (tid < 15) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < N_MONO; ++i) s += zs[tid * N_MONO + i] * M[i];
    out[2 + tid] = -grad_scale * s;
  } else if (tid == 15) {
    double l = 0.0;
    for (int i = 0; has_loss && i < GRAD_LOSS_BLOCKS; ++i) l += sums[(size_t)T * N_MONO + i];
    out[0] = l;
    out[1] = -grad_scale * (0.5 * (double)N * (double)N) * (W[3] + W[5]);
  }
}

hipError_t launch_grad_finish(int T, int N, int nblk, const double* mono_partials, const double* loss_partials,
                              int n_loss, const double* alpha_over_z, const double* zmat, double grad_scale,
                              double* sums, double* out, hipStream_t s) {
  const int nl = n_loss > 0 ? GRAD_LOSS_BLOCKS : 0;
  hipLaunchKernelGGL(k_grad_frames, dim3(T + nl), dim3(GF_THREADS), 0, s, T, nblk, mono_partials, loss_partials,
                     n_loss, grad_scale, sums, out);
  hipLaunchKernelGGL(k_grad_finish, dim3(1), dim3(GF_THREADS), 0, s, T, N, sums, alpha_over_z, zmat, grad_scale,
                     nl, out);
  return hipGetLastError();
}

}  // namespace ssoct
