// Vector kernels of the implicit (Newton-Krylov) time step.  Every
// reduction has a fixed assignment of elements to work-groups and a fixed
// summation order for a given length, so results are bitwise reproducible.
// The multi-dot and multi-axpy kernels take two consecutive elements per
// access: their FP64 vectors must be 16-byte aligned, FP32 basis vectors
// (base and stride) 8-byte aligned.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>

namespace dgbgk {

// Most vectors one multi-dot or multi-axpy call takes.
constexpr int kMaxBasis = 72;

// out = a x + b y + c z; a term is skipped when its pointer is null.  out may
// alias any input (element-wise update).
hipError_t launch_lincomb(size_t n, double a, const double *x, double b, const double *y, double c,
                          const double *z, double *out, hipStream_t stream);

// Doubles of scratch that launch_multi_dot needs for length n and nv vectors.
size_t multi_dot_scratch(size_t n, int nv);

// result[k] = V_k . w for k < nv, V_k = V + k * stride (nv <= kMaxBasis).
// scratch holds multi_dot_scratch(n, nv) doubles; result is device memory.  host,
// when not null: pinned host memory that receives the results as well.
hipError_t launch_multi_dot(size_t n, int nv, const double *V, size_t stride, const double *w,
                            double *scratch, double *result, hipStream_t stream, double *host = nullptr);

// out = scale (w + alpha sum_{k < nv} coef[k] V_k), coef in device memory
// (nv <= kMaxBasis); out may alias w.  t, when not null, receives y + e out.
hipError_t launch_multi_axpy(size_t n, int nv, const double *V, size_t stride, const double *coef,
                             double alpha, const double *w, double scale, double *out,
                             hipStream_t stream, const double *y = nullptr, double e = 0.0,
                             double *t = nullptr);

// w -= sum_{k < nv} coef[k] V_k, then result[k] = V_k . w for k < nv and
// result[nv] = w . w, for 1 <= nv <= kOrthBasis; w is none of the V_k.  scratch
// as for launch_multi_dot(n, nv + 1).
constexpr int kOrthBasis = 8;
hipError_t launch_multi_orth(size_t n, int nv, const double *V, size_t stride, const double *coef, double *w,
                             double *scratch, double *result, hipStream_t stream, double *host = nullptr);

// The last update of a Gram-Schmidt pass (1 or 2) before the host has seen its
// products: as launch_multi_axpy(V, h, alpha = -1, w, scale, w, y, e, t) with
// h[0..nv) the projections of w, h[nv] = |w|^2 and scale = orth_scale(pass, nv, h).
hipError_t launch_multi_orth_scaled(size_t n, int pass, int nv, const double *V, size_t stride, const double *h,
                                    double *w, hipStream_t stream, const double *y, double e, double *t);

// 1 / |w - V h| = (|w|^2 - |h|^2)^(-1/2); 1 where pass 1 cancels more than half
// of |w|^2 (a second pass follows) or nothing is left.  Host and device take the
// same branch: no product is contracted into a sum.
__host__ __device__ inline double orth_scale(int pass, int nv, const double *h) {
#pragma clang fp contract(off)
  double hh = 0.0;
  for (int k = 0; k < nv; ++k) hh += h[k] * h[k];
  const double d = h[nv] - hh;
  return d > (pass == 1 ? 0.5 * h[nv] : 0.0) ? 1.0 / sqrt(d) : 1.0;
}

// The same operations with the Krylov basis V stored in FP32 (w, coef and
// out stay FP64).  lincomb_mixed: out = a x + b y + c z with y in FP32.
hipError_t launch_lincomb_mixed(size_t n, double a, const double *x, double b, const float *y,
                                double c, const double *z, double *out, hipStream_t stream);

// result[k] = V_k . w for k < nv and result[nv] = w . w (nv + 1 <= kMaxBasis);
// scratch holds multi_dot_scratch(n, nv + 1) doubles.
hipError_t launch_multi_dot32(size_t n, int nv, const float *V, size_t stride, const double *w,
                              double *scratch, double *result, hipStream_t stream);

// out = scale (w + alpha sum_{k < nv} coef[k] V_k); out32, when not null,
// receives out rounded to FP32, and t, when neither is null, y + e out32.  out
// may alias w.
hipError_t launch_multi_axpy32(size_t n, int nv, const float *V, size_t stride, const double *coef,
                               double alpha, const double *w, double scale, double *out,
                               float *out32, hipStream_t stream, const double *y = nullptr, double e = 0.0,
                               double *t = nullptr);

}  // namespace dgbgk
