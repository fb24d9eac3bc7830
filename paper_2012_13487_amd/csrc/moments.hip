// Density and velocity at every node of an element-major state.
#include "moments.hpp"

namespace dgbgk {

namespace {

constexpr int kThreads = 256;
// A launch holds fewer than 2^32 threads along x: of more elements than this
// the work-groups take several.
constexpr int kMaxGroups = (1 << 24) - 1;

// A work-group per element: its Q Np values are read once in memory order, H
// velocities at a time (H Np threads), so that each thread keeps its node; the
// H partial sums meet in LDS.  Bound by that read.  A thread per node that walks
// all velocities takes a chain of Q loads instead, with too few threads to hide
// it: 72x72 elements, p = 2, 256 velocities: 97 us for one FP64 state (and 36 us
// before it to form f_ref + g), now 25 us, and 31 us from f_ref and g together.
template <bool FD, bool FS>
__global__ __launch_bounds__(kThreads) void node_moments_kernel(const double *fd, const float *fs, double offset,
                                                               const double *vel, int K, int Np, int Q, int H,
                                                               double *rho, double *ux, double *uy) {
  __shared__ double red[3][kThreads];
  const int t = threadIdx.x, h = t / Np, n = t - h * Np;
  for (int k = blockIdx.x; k < K; k += gridDim.x) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (h < H) {
      const size_t base = (size_t)k * Q * Np + n;
#pragma unroll 4
      for (int q = h; q < Q; q += H) {
        const size_t i = base + (size_t)q * Np;
        double v = FD ? fd[i] : 0.0;
        if (FS) v += (double)fs[i];
        if (offset != 0.0) v += vel[2 * Q + q] * offset;
        s0 += v;
        s1 += vel[q] * v;
        s2 += vel[Q + q] * v;
      }
    }
    if (k != (int)blockIdx.x) __syncthreads();  // (the sums of the element before have been read)
    red[0][t] = s0;
    red[1][t] = s1;
    red[2][t] = s2;
    __syncthreads();
    if (t < Np) {
      s0 = s1 = s2 = 0.0;
#pragma unroll 4
      for (int g = 0; g < H; ++g) {
        s0 += red[0][g * Np + t];
        s1 += red[1][g * Np + t];
        s2 += red[2][g * Np + t];
      }
      const size_t o = (size_t)k * Np + t;
      rho[o] = s0;
      ux[o] = s1 / s0;
      uy[o] = s2 / s0;
    }
  }
}

}  // namespace

hipError_t launch_node_moments(const double *fd, const float *fs, double offset, const double *vel, int K, int Np,
                               int Q, double *rho, double *ux, double *uy, hipStream_t st) {
  if (Np < 1 || Np > kThreads || (!fd && !fs)) return hipErrorInvalidValue;
  const int H = kThreads / Np < Q ? kThreads / Np : Q;
  const dim3 grid((unsigned)(K < kMaxGroups ? K : kMaxGroups)), block(kThreads);
  if (fd && fs)
    hipLaunchKernelGGL((node_moments_kernel<true, true>), grid, block, 0, st, fd, fs, offset, vel, K, Np, Q, H,
                       rho, ux, uy);
  else if (fd)
    hipLaunchKernelGGL((node_moments_kernel<true, false>), grid, block, 0, st, fd, fs, offset, vel, K, Np, Q, H,
                       rho, ux, uy);
  else
    hipLaunchKernelGGL((node_moments_kernel<false, true>), grid, block, 0, st, fd, fs, offset, vel, K, Np, Q, H,
                       rho, ux, uy);
  return hipGetLastError();
}

}  // namespace dgbgk
