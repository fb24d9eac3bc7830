// Row kernels of FP64 (rows_kernel.hpp).
#include "rows_kernel.hpp"

namespace dgbgk {

RowPlan row_plan(int p, int64_t K, int Q, int size, bool ref) {
  RowPlan r;
  if (p < 1 || p > kRowMaxP || Q < kRowMinQ || K < 1) return r;
  const int64_t most_waves = (((int64_t)1 << 32) - 1) / 64;  // a launch holds fewer than 2^32 threads along x
  const int n1 = p + 1, np = n1 * n1, pr = row_period(np, size);
  const int fit = row_elements_max(np, size, Q);
  if (fit >= 1) {
    // whole elements in the wavefront, fewer of them while the mesh leaves
    // compute units without one
    r.kind = 2;
    r.ew = fit < 4 ? fit : 4;
    while (r.ew > 1 && (K + r.ew - 1) / r.ew < 512) r.ew = (r.ew + 1) / 2;
    if ((K + r.ew - 1) / r.ew > most_waves) return RowPlan{};
    r.nw = 1;
    r.nblk = (int)((K + r.ew - 1) / r.ew);
    r.lds = (size_t)row_elements_bytes(n1, size, ref, r.ew);
    return r;
  }
  // an element's rows in 64s, dealt to work-groups of up to four wavefronts
  // (more resident at a time than with one large work-group per element); the
  // split with the fewest idle wavefronts, and of these the fewest tiles, whose
  // partial sums every work-group of the element reads
  const int nch = (Q + (Q % pr == 0 ? 0 : pr - 1) + 63) / 64;
  int best = 1 << 30;
  for (int nw = 2; nw <= 4; ++nw) {
    const int nt = (nch + nw - 1) / nw;
    if (nt <= kMaxPartialTiles && nt * nw <= best) {
      best = nt * nw;
      r.nw = nw;
      r.nt = nt;
    }
  }
  if (best == 1 << 30 || K * r.nw > most_waves) return RowPlan{};
  r.kind = 1;
  r.ew = 1;
  r.nblk = (int)K;
  const int factors = (np * node_values_of(size, ref) * size + 15) / 16 * 16 + 4 * n1 * 8;
  const int sums = r.nw * row_sum_parts(np, size) * 3 * np * 8;
  r.lds = (size_t)r.nw * (row_wave_bytes(np, size) + 64 * 16) + factors + sums;
  return r;
}

hipError_t launch_rows(int p, int kind, const RowArgs<double> &a, size_t lds, hipStream_t st) {
  using namespace rows;
  switch (p) {
    case 1: return launch_kind<1, double, false>(kind, a, lds, st);
    case 2: return launch_kind<2, double, false>(kind, a, lds, st);
    case 3: return launch_kind<3, double, false>(kind, a, lds, st);
    case 4: return launch_kind<4, double, false>(kind, a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

namespace {

// Thread: one of the 3 Np moment rates of an element.
__global__ __launch_bounds__(256) void rate_max_kernel(const double *part, size_t KN3, int K, int np, int nt,
                                                       double scale, unsigned long long *result) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  double m = 0.0;
  if (i < KN3) {
    const size_t k = i / (3 * np), o = i - k * 3 * np;
    double s = 0.0;
    for (int t = 0; t < nt; ++t) s += part[((size_t)t * K + k) * 7 * np + o];
    m = fabs(s) * scale;
  }
  rows::max_out(m, result);
}

}  // namespace

hipError_t launch_rate_max(const double *part, int K, int Np, int nt, double scale, unsigned long long *result,
                           hipStream_t st) {
  const size_t n = (size_t)K * 3 * Np;
  hipLaunchKernelGGL(rate_max_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, n, K, Np, nt,
                     scale, result);
  return hipGetLastError();
}

hipError_t launch_rows_sums(int p, const RowArgs<double> &a, size_t lds, hipStream_t st) {
  using namespace rows;
  switch (p) {
    case 1: return launch_one<kKindSums, 1, double, 0, false>(a, lds, st);
    case 2: return launch_one<kKindSums, 2, double, 0, false>(a, lds, st);
    case 3: return launch_one<kKindSums, 3, double, 0, false>(a, lds, st);
    case 4: return launch_one<kKindSums, 4, double, 0, false>(a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch_rows(int p, int stage, const RowArgs<double> *descs, const int2 *items, int nitems,
                             size_t lds, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  return rows::launch_batch_any<double, false>(p, stage, descs, items, nitems, lds, st);
}

}  // namespace dgbgk
