// Row kernels (rows_kernel.hpp): sizes, launch plan and launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "kernels.hpp"

namespace dgbgk {

constexpr int kRowMaxN1 = 5;
constexpr int kRateSums = 5;  // the stage of launch_rows that reduces the moment rates of L(f_s) only
constexpr int kJacobian = 6;  // FP64: out = fn + c_out (L(f_s) - f1)
constexpr int kRowMaxP = 4;  // a row's values and rates live in registers
constexpr int kRowStripMin = 1024;  // work-groups from which their order matters to the caches
constexpr int kRowMinQ = 8;  // fewer velocities leave most lanes of a wavefront without a row

// Rows after which 16-byte accesses over consecutive rows of np values repeat
// their nodes.
__host__ __device__ constexpr int row_period(int np, int size) {
  const int vw = 16 / size;
  return np % vw == 0 ? 1 : (np % 2 == 0 ? vw / 2 : vw);
}
// LDS stride of a row, in values: odd node counts keep the memory image (an
// odd stride has no bank conflicts); even ones are padded, or permuted, so that
// the 16-byte accesses of 16 consecutive rows fall on distinct banks.
__host__ __device__ constexpr bool row_swizzled(int np, int size) { return np * size == 128; }
__host__ __device__ constexpr int row_stride(int np, int size) {
  return np % 2 || row_swizzled(np, size) ? np : size == 8 ? np + 2 : np == 4 ? 4 : np + 4;
}
__host__ __device__ constexpr int row_tile_bytes(int np, int size) { return 64 * row_stride(np, size) * size; }
// Column sums of a wavefront at odd node counts, which go through its tile: all
// three of 1, e_x, e_y at once where they fit, and into how many parts.
__host__ __device__ constexpr bool row_sums_at_once(int np, int size) {
  const int vw = 16 / size, pr = row_period(np, size), lanes = 64 / (pr * np / vw) * (pr * np / vw);
  return 3 * lanes * vw * 8 <= row_tile_bytes(np, size);
}
__host__ __device__ constexpr int row_sum_parts(int np, int size) {
  if (np % 2 == 0) return 1;
  const int o = row_sums_at_once(np, size) ? 3 * np : np;
  return 64 / o > 0 ? 64 / o : 1;
}
// A wavefront's tile in LDS (it also takes 64 doubles of wall sums, and the
// column sums of one component).
__host__ __device__ constexpr int row_wave_bytes(int np, int size) {
  const int vw = 16 / size, pr = row_period(np, size), lanes = 64 / (pr * np / vw) * (pr * np / vw);
  const int sums = np % 2 ? lanes * vw * 8 : 512, tile = row_tile_bytes(np, size);
  return tile > sums ? tile : sums;
}
// Node factors kept per node, in values.
__host__ __device__ constexpr int node_values_of(int size, bool ref) { return size == 8 ? 4 : ref ? 12 : 8; }
__host__ __device__ constexpr int row_node_stride(int np, int size, bool ref) {
  return np * node_values_of(size, ref) + (size == 8 ? 2 : 4);  // (an element's, padded against bank conflicts)
}
// LDS of a wavefront that owns ew elements: its tile, the rows' velocities, the
// elements' node factors and wall densities.
__host__ __device__ constexpr int row_elements_bytes(int n1, int size, bool ref, int ew) {
  return row_wave_bytes(n1 * n1, size) + 64 * 16 + (ew * row_node_stride(n1 * n1, size, ref) * size + 15) / 16 * 16 +
         (ew * 4 * n1 * 8 + 15) / 16 * 16;
}
// Elements of q velocities whose rows fit a wavefront's 64 (after the lead).
__host__ __device__ constexpr int row_elements_max(int np, int size, int q) {
  const int pr = row_period(np, size);
  return (q % pr == 0 ? 64 : 64 - pr + 1) / q;
}

struct RowPlan {
  int kind = 0;  // 0: none; 1: an element's velocities in 64s, moments handed over; 2: moments in the wavefront
  int nw = 0;    // wavefronts per work-group, 64 velocities each (kind 1)
  int nt = 1;    // velocity tiles (work-groups) per element (kind 1)
  int ew = 0;    // elements per wavefront (kind 2)
  int nblk = 0;  // work-groups (one wavefront each, kind 2)
  size_t lds = 0;
};

// x / d for 0 <= x < 2^31 by a reciprocal (ceil(2^32 / d)) and one correction.
struct RowDivisor {
  unsigned d, inv;
};
inline RowDivisor row_divisor(int d) {
  const unsigned long long u = (unsigned long long)d;
  return {(unsigned)d, (unsigned)((((unsigned long long)1 << 32) + u - 1) / u)};
}

// One launch of the row kernels (T: double, or float for the FP32 storage
// forms), held to what they read: the arguments reach a wavefront 64 bytes at a
// time, each a miss of the scalar cache at the start of a launch.
template <typename T>
struct RowArgs {
  const double *vel;   // [3][Q]: e_x, e_y, w
  const T *fs;         // stage input
  RowDivisor dnx;      // elements per mesh row
  int nx, ny, K, Q;
  int kind, nw, nt, ew, nblk, lds;  // the plan
  int strip_w, strips, strip_last, strip_row;  // strip order: work-groups per strip, whole strips, the
  RowDivisor dstrip, dw, dlast;                // last one's width, work-groups per mesh row
  RowDivisor dnt;
  int wall_mask, periodic_x, periodic_y;
  int stream_nt;       // 1: the streams move with non-temporal hints
  const double *pin;   // moment sums of fs per velocity tile and element [tile][K][7][Np] (kind 1)
  double *pout;        // those of out
  const double *feqb;  // [4][Q]: f^eq_q(1, u_b) of each side's wall velocity
  const T *fn;         // state at the start of the step
  T *out;
  const T *f1, *f2;    // FP64: the states of stages 2 and 3, read by the last stage
  T *acc;              // FP32 storage: the RK4 accumulator
  const float *rref;   // reference form: L(f_r), and rho, u of f_r per node ([3][K Np])
  const double *mref;
  T rx, sy;            // 2/hx, 2/hy
  T lift[kRowMaxN1];   // M1^{-1} e_0: lift of a flux on the left / bottom face
  T D1[(kRowMaxN1 * kRowMaxN1 + 1) / 2];  // first half of the 1-D differentiation matrix (the rest mirrors it)
  T theta_inv, half_theta2_inv, inv_tau;
  T c_acc, c_out;      // RK4 coefficients of this stage (times dt)
  double half_theta_inv;
  double wall_den_inv[4];
  double rho_ref;      // FP32 storage: g = f - w rho_ref, and the moments of that part
  double mconst[7];
  double resid_scale;  // kRateSums: the largest scaled moment rate goes to *result (one velocity tile), or the
  unsigned long long *result;  // sums to pout (several; launch_rate_max)
  int stage;           // 0: out = L(f_s); 1..4: classical RK4 stage; kRateSums; kJacobian
};

// The plan for a problem of order p with Q velocities and K elements; value
// size 8 (FP64) or 4 (FP32 storage; ref: the reference form).
RowPlan row_plan(int p, int64_t K, int Q, int size, bool ref);

// The plan's fields of the arguments (a.nx set).
template <typename T>
void row_plan_args(const RowPlan &r, RowArgs<T> &a) {
  a.kind = r.kind;
  a.nw = r.nw;
  a.nt = r.nt;
  a.ew = r.ew;
  a.nblk = r.nblk;
  a.lds = (int)r.lds;
  a.dnx = row_divisor(a.nx);
  a.dnt = row_divisor(r.nt);
  // strips 16 elements wide, where the work-groups tile whole mesh rows
  const int per = r.kind == 2 ? r.ew : 1;
  a.strip_w = a.strips = a.strip_last = a.strip_row = 0;
  a.dstrip = a.dw = a.dlast = row_divisor(1);
  if (a.nx % per || r.nblk < kRowStripMin) return;
  const int bpr = a.nx / per, w = 16 / per;
  a.strip_w = w;
  a.strips = bpr / w;
  a.strip_last = bpr % w ? bpr % w : w;
  a.strip_row = bpr;
  a.dstrip = row_divisor(w * (r.nblk / bpr));
  a.dw = row_divisor(w);
  a.dlast = row_divisor(a.strip_last);
}

// One stage.
hipError_t launch_rows(int p, int kind, const RowArgs<double> &a, size_t lds, hipStream_t st);
hipError_t launch_rows32(int p, int kind, int ref, const RowArgs<float> &a, size_t lds, hipStream_t st);

// *result = max(*result, scale |moment rate|) from the tiles' rate sums in part.
hipError_t launch_rate_max(const double *part, int K, int Np, int nt, double scale, unsigned long long *result,
                           hipStream_t st);

// The moment sums of the state a.fs into a.pout (kind 1), by the same lanes in
// the same order as the stages sum their outputs.
hipError_t launch_rows_sums(int p, const RowArgs<double> &a, size_t lds, hipStream_t st);
hipError_t launch_rows_sums32(int p, const RowArgs<float> &a, size_t lds, hipStream_t st);

// A plan's work-groups of 256 threads in a batch: two elements each where two
// wavefronts take one, else one; four wavefronts' runs of elements.
inline int row_items(const RowPlan &r) {
  const int per = r.kind == 2 ? 4 : r.nw == 2 ? 2 : 1;
  return (r.nblk * r.nt + per - 1) / per;
}
inline size_t row_item_lds(const RowPlan &r) { return (r.kind == 2 ? 4 : r.nw == 2 ? 2 : 1) * r.lds; }

// Batched stages: one work-group of 256 threads per item (problem, work-group;
// row_items of them per problem), descriptors as in launch_batch_stage, problems
// of order p; lds: the largest row_item_lds.
hipError_t launch_batch_rows(int p, int stage, const RowArgs<double> *descs, const int2 *items, int nitems,
                             size_t lds, hipStream_t st);
hipError_t launch_batch_rows32(int p, int ref, int stage, const RowArgs<float> *descs, const int2 *items,
                               int nitems, size_t lds, hipStream_t st);

}  // namespace dgbgk
