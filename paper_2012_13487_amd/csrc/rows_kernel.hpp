// Row kernels: the RK stage by wavefronts that each own a run of velocity rows.
//
// A velocity row is the Np nodal values of one velocity in one element; the
// rows of an element are consecutive in memory.  One wavefront takes 64 rows
// at a time: it copies them into a tile of its own in LDS with coalesced
// 16-byte loads, evaluates L(f) with one row per lane in registers (volume
// term by sum factorisation, upwind jumps, collision), puts the result back
// into the tile and makes the RK update with coalesced 16-byte accesses.  The
// tile belongs to one wavefront, so nothing in this chain waits for another
// one: the wavefronts of a compute unit drift apart and their loads, row
// arithmetic and stores overlap, where the kernels that stage a whole element
// per work-group pass four barriers with every wavefront in the same phase.
//
// The node moments the collision needs are sums over all velocities:
//  * handed over (more velocities than a wavefront has rows): one element, and
//    up to 256 of its velocities, per work-group; the update pass also sums 1,
//    e_x, e_y (and, at walls, the outgoing normal speeds) times its outputs per
//    node, and the next stage reads the sums (7 Np doubles per element) before
//    its rows;
//  * in the wavefront (an element's rows fit a wavefront): the wavefront owns
//    whole elements and sums over the velocities from its tile.
//
// Bound: HBM.  The row chain needs 13 loads in flight per lane at p = 4 and
// LDS for the tile (12.8 KB per wavefront in FP64), which leaves 9 to 20
// wavefronts per compute unit.
//
// Odd node counts (p = 2, 4): 16-byte accesses straddle rows.  Two rows (FP64)
// or four (FP32) are a whole number of accesses, so a wavefront's rows are
// counted from a row whose address is a multiple of 16 bytes (the lead: up to
// three rows of the element before, loaded and ignored) and the lanes of an
// access group keep their nodes from one pass to the next.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "rows.hpp"

namespace dgbgk {
namespace rows {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct VecOf;
template <>
struct VecOf<double> { typedef d2 type; };
template <>
struct VecOf<float> { typedef f4 type; };

template <int P, typename T>
struct RowShape {
  static constexpr int N1 = P + 1, NP = N1 * N1;
  static constexpr int VW = 16 / sizeof(T);             // values per access
  static constexpr int PR = row_period(NP, sizeof(T));  // rows after which accesses repeat their nodes
  static constexpr int RA = PR * NP / VW;               // accesses in that many rows
  static constexpr int G = 64 / RA;                     // access groups of a wavefront
  static constexpr int RPI = G * PR;                    // rows per pass of the update
  static constexpr int NIT = (64 + RPI - 1) / RPI;      // passes over 64 rows
  static constexpr int S = row_stride(NP, sizeof(T));   // LDS row stride
  static constexpr bool SWZ = row_swizzled(NP, sizeof(T));
  static constexpr bool LIN = S == NP && !SWZ;          // the tile is an image of memory
  static constexpr int NLD = (64 * NP / VW + 63) / 64;  // accesses per lane of a tile
  // Place of value n of row r in the tile.  Rows of 128 bytes (FP64, p = 3) are
  // not padded (four work-groups per compute unit instead of three): their
  // 16-byte pieces are permuted by the row instead, so that 16 consecutive rows
  // read at one node fall on distinct banks.
  __device__ static __forceinline__ int at(int r, int n) {
    if constexpr (SWZ) return r * NP + (((n / VW) ^ ((r >> 1) & 7)) * VW) + n % VW;
    return r * S + n;
  }
};

// LDS accesses of one wavefront complete in order; this keeps the compiler
// from moving them across the hand-over between lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Global accesses at a wave-uniform base plus a 32-bit byte offset per lane, so
// that an access needs one offset register rather than a 64-bit address.
template <bool NT, typename V, typename T>
__device__ __forceinline__ V ld_stream(const T *base, unsigned bytes) {
  const V *p = reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + bytes);
  if constexpr (NT) return __builtin_nontemporal_load(p);
  return *p;
}
template <bool NT, typename V, typename T>
__device__ __forceinline__ void st_stream(T *base, unsigned bytes, const V &v) {
  V *p = reinterpret_cast<V *>(reinterpret_cast<char *>(base) + bytes);
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

__device__ __forceinline__ int quotient(int x, const RowDivisor &d) {
  if (d.d == 1) return x;
  const int q = (int)__umulhi((unsigned)x, d.inv);
  return (unsigned)q * d.d > (unsigned)x ? q - 1 : q;
}

// Mesh place of the e-th element after the one at (ex0, ey0), e <= 3.
template <typename A>
__device__ __forceinline__ void step_place(int ex0, int ey0, int e, const A &a, int &ex, int &ey) {
  ex = ex0 + e;
  ey = ey0;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const bool wrap = ex >= a.nx;
    ex -= wrap ? a.nx : 0;
    ey += wrap ? 1 : 0;
  }
}

template <typename A>
__device__ __forceinline__ int row_neighbour(int ex, int ey, int k, int face, const A &a) {
  switch (face) {
    case 0: return ey > 0 ? k - a.nx : (a.periodic_y ? k + a.nx * (a.ny - 1) : -1);
    case 1: return ex < a.nx - 1 ? k + 1 : (a.periodic_x ? k - (a.nx - 1) : -1);
    case 2: return ey < a.ny - 1 ? k + a.nx : (a.periodic_y ? k - a.nx * (a.ny - 1) : -1);
    default: return ex > 0 ? k - 1 : (a.periodic_x ? k + (a.nx - 1) : -1);
  }
}

// ---- node factors of the collision, one set per node in LDS ----------------

// Floating values per node: FP64 u_x, u_y, rho, 1 - |u|^2 / (2 theta); FP32
// storage u_x, u_y, rho, rho - rho_ref, |u|^2 / (2 theta); reference form the
// nine factors of the difference of equilibria.
template <typename T, bool REF>
constexpr int node_values() { return node_values_of(sizeof(T), REF); }

__device__ __forceinline__ void node_factors(const RowArgs<double> &a, const double (&sm)[3], const double *,
                                             double *m) {
  const double rho = sm[0], ux = sm[1] / rho, uy = sm[2] / rho;
  m[0] = ux;
  m[1] = uy;
  m[2] = rho;
  m[3] = 1.0 - (ux * ux + uy * uy) * a.half_theta_inv;
}

template <bool REF>
__device__ __forceinline__ void node_factors32(const RowArgs<float> &a, double (&sm)[3], const double *ref,
                                               float *m) {
  if constexpr (REF) {
    // moments of g are the increments over the reference's (FP64)
    const double rr = ref[0], urx = ref[1], ury = ref[2];
    const double drho = sm[0], rho = rr + drho;
    const double ux = (rr * urx + sm[1]) / rho, uy = (rr * ury + sm[2]) / rho;
    const double dux = ux - urx, duy = uy - ury;
    const double h1 = a.half_theta_inv, th_inv = 2.0 * h1, h2 = h1 * th_inv;
    // rho |u|^2 - rho_r |u_r|^2 = drho |u|^2 + rho_r (u + u_r).(u - u_r)
    const double dq = drho * (ux * ux + uy * uy) + rr * ((ux + urx) * dux + (uy + ury) * duy);
    m[0] = (float)(drho - dq * h1);
    m[1] = (float)(sm[1] * th_inv);
    m[2] = (float)(sm[2] * th_inv);
    m[3] = (float)urx;
    m[4] = (float)ury;
    m[5] = (float)dux;
    m[6] = (float)duy;
    m[7] = (float)(drho * h2);
    m[8] = (float)(rho * h2);
  } else {
    const double rho = sm[0] + a.mconst[0], ux = (sm[1] + a.mconst[1]) / rho,
                 uy = (sm[2] + a.mconst[2]) / rho;
    m[0] = (float)ux;
    m[1] = (float)uy;
    m[2] = (float)rho;
    m[3] = (float)(rho - a.rho_ref);
    m[4] = (float)((ux * ux + uy * uy) * a.half_theta_inv);
  }
}

template <bool REF>
__device__ __forceinline__ void node_factors_t(const RowArgs<double> &a, double (&sm)[3], const double *ref,
                                               double *m) {
  node_factors(a, sm, ref, m);
}
template <bool REF>
__device__ __forceinline__ void node_factors_t(const RowArgs<float> &a, double (&sm)[3], const double *ref,
                                               float *m) {
  node_factors32<REF>(a, sm, ref, m);
}

// Constant part of the outgoing wall flux of side fc in the stored state.
template <bool REF>
__device__ __forceinline__ double wall_const(const RowArgs<double> &, int) { return 0.0; }
template <bool REF>
__device__ __forceinline__ double wall_const(const RowArgs<float> &a, int fc) {
  return REF ? 0.0 : a.mconst[3 + fc];
}

// ---- L(f) of one row in registers -------------------------------------------

// D1[i][m] on Gauss-Lobatto nodes, which are symmetric: D1[P-i][P-m] =
// -D1[i][m] (and the lift of the far face mirrors the near one's), so half the
// table sits in scalar registers.
template <int N1, typename A>
__device__ __forceinline__ auto d1_entry(const A &a, int i, int m) {
  const int at = i * N1 + m, mirror = N1 * N1 - 1 - at;
  return at <= mirror ? a.D1[at] : -a.D1[mirror];
}

// Volume term and upwind jumps: kk = -(e . grad f) + lifted jumps; px, py are
// the exterior traces of the inflow faces.  A velocity along a face has a zero
// jump coefficient there.
template <int P, typename A, typename T>
__device__ __forceinline__ void row_transport(const A &a, const T (&f)[(P + 1) * (P + 1)], T cx, T cy,
                                              const T (&px)[P + 1], const T (&py)[P + 1],
                                              T (&kk)[(P + 1) * (P + 1)]) {
  constexpr int N1 = P + 1;
  const T ax = -cx * a.rx, ay = -cy * a.sy;
#pragma unroll
  for (int j = 0; j < N1; ++j)
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      T dr = 0, ds = 0;
#pragma unroll
      for (int m = 0; m < N1; ++m) {
        dr += d1_entry<N1>(a, i, m) * f[m + N1 * j];
        ds += d1_entry<N1>(a, j, m) * f[i + N1 * m];
      }
      kk[i + N1 * j] = ax * dr + ay * ds;
    }
  const bool right = cx > 0, up = cy > 0;  // inflow at the left / bottom face
  const T wx = a.rx * (right ? -cx : cx), wy = a.sy * (up ? -cy : cy);
  T lx[N1], ly[N1];
#pragma unroll
  for (int m = 0; m < N1; ++m) {
    lx[m] = right ? a.lift[m] : a.lift[P - m];
    ly[m] = up ? a.lift[m] : a.lift[P - m];
  }
#pragma unroll
  for (int jj = 0; jj < N1; ++jj) {
    const T J = wx * ((right ? f[N1 * jj] : f[N1 * jj + P]) - px[jj]);
#pragma unroll
    for (int ii = 0; ii < N1; ++ii) kk[ii + N1 * jj] += lx[ii] * J;
  }
#pragma unroll
  for (int ii = 0; ii < N1; ++ii) {
    const T J = wy * ((up ? f[ii] : f[ii + N1 * P]) - py[ii]);
#pragma unroll
    for (int jj = 0; jj < N1; ++jj) kk[ii + N1 * jj] += ly[jj] * J;
  }
}

// kk += (f^eq - f) / tau at every node (node factors mm).
template <int P, bool REF>
__device__ __forceinline__ void row_collide(const RowArgs<double> &a, const double *mm, double cx, double cy,
                                            double wq, const double (&f)[(P + 1) * (P + 1)],
                                            double (&kk)[(P + 1) * (P + 1)]) {
#pragma unroll
  for (int nn = 0; nn < (P + 1) * (P + 1); ++nn) {
    const d2 u = *reinterpret_cast<const d2 *>(mm + 4 * nn), m = *reinterpret_cast<const d2 *>(mm + 4 * nn + 2);
    const double eu = cx * u[0] + cy * u[1];
    const double feq = wq * m[0] * (m[1] + eu * (a.theta_inv + eu * a.half_theta2_inv));
    kk[nn] += (feq - f[nn]) * a.inv_tau;
  }
}
template <int P, bool REF>
__device__ __forceinline__ void row_collide(const RowArgs<float> &a, const float *mm, float cx, float cy,
                                            float wq, const float (&f)[(P + 1) * (P + 1)],
                                            float (&kk)[(P + 1) * (P + 1)]) {
  constexpr int MS = node_values<float, REF>();
#pragma unroll
  for (int nn = 0; nn < (P + 1) * (P + 1); ++nn) {
    const float *m = mm + MS * nn;
    float dev;
    if constexpr (REF) {
      // f^eq / w = rho + e.j/theta + [rho (e.u)^2 / theta - rho |u|^2] / (2 theta):
      // a = e.u_r, b = e.(u - u_r); rho (e.u)^2 - rho_r a^2 = drho a^2 + rho b (2a + b)
      const float av = cx * m[3] + cy * m[4], bv = cx * m[5] + cy * m[6];
      dev = wq * (m[0] + cx * m[1] + cy * m[2] + m[7] * av * av + m[8] * bv * (2.0f * av + bv));
    } else {
      // w [(rho - rho_ref) + rho (e.u/theta + (e.u)^2/(2 theta^2) - |u|^2/(2 theta))]
      const f4 m4 = *reinterpret_cast<const f4 *>(m);
      const float usq = m[4];
      const float eu = cx * m4[0] + cy * m4[1];
      dev = wq * (m4[3] + m4[2] * (eu * (a.theta_inv + eu * a.half_theta2_inv) - usq));
    }
    kk[nn] += (dev - f[nn]) * a.inv_tau;
  }
}

// What the row phase leaves in the tile: FP64 stages 1 and 4 form f + dt/2 k
// there (see update_value); everything else k.
template <int MODE, int NP>
__device__ __forceinline__ void row_result(const RowArgs<double> &a, const double (&f)[NP], double (&kk)[NP]) {
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    if (MODE == 1) kk[c] = f[c] + a.c_out * kk[c];
    if (MODE == 4) kk[c] = f[c] + 3.0 * a.c_acc * kk[c];
  }
}
template <int MODE, int NP>
__device__ __forceinline__ void row_result(const RowArgs<float> &, const float (&)[NP], float (&)[NP]) {}

// ---- the RK update ------------------------------------------------------------

// FP64, classical RK4 from the stage states (f_1 - f_n = dt/2 k_1, f_2 - f_n =
// dt/2 k_2, f_3 - f_n = dt k_3), so that no accumulator is written: 16, 24, 24
// and 40 bytes per value in stages 1 to 4.
//   MODE 0: o = k (kRateSums: o is summed, not stored)      kJacobian: o = x + c (k - y)
//   MODE 1: o = kv = f_n + dt/2 k      2: o = x + c k  (x = f_n)
//   MODE 4: o = x + [(y - x) + 2 (z - x) + (kv - x)] / 3, kv = f_3 + dt/2 k  (x = f_n, y = f_1,
//           z = f_2; the differences are small, so the state is rounded once)
// FP32, increment form (the state is rounded once per step): d = sum b_i dt k_i
//   MODE 1: d = dt/6 k, o = x + dt/2 k      2: d += c k, o = x + c' k      4: o = x + (d + dt/6 k)
// Whether a mode hands on the sums of its outputs (kind 1).
constexpr bool row_sums_mode(int mode) { return mode != 0 && mode != kJacobian; }

template <typename T, int MODE>
struct Streams {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr bool X = F64 ? (MODE == 2 || MODE == 4 || MODE == kJacobian) : MODE != 0 && MODE != kRateSums;
  static constexpr bool Y = F64 ? (MODE == 4 || MODE == kJacobian) : (MODE == 2 || MODE == 4);
  static constexpr bool Z = F64 && MODE == 4;
  static constexpr bool ACC = !F64 && (MODE == 1 || MODE == 2);
};
template <int MODE>
__device__ __forceinline__ double update_value(double kv, double x, double y, double z, double,
                                               double co, double &) {
  if (MODE == 2) return x + co * kv;
  if (MODE == kJacobian) return x + co * (kv - y);
  if (MODE == 4) return x + ((y - x) + 2.0 * (z - x) + (kv - x)) * (1.0 / 3.0);
  return kv;
}
template <int MODE>
__device__ __forceinline__ float update_value(float kv, float x, float y, float, float ca, float co,
                                              float &an) {
  if (MODE == 0 || MODE == kRateSums) return kv;
  if (MODE == 1) { an = ca * kv; return x + co * kv; }
  if (MODE == 2) { an = y + ca * kv; return x + co * kv; }
  return x + (y + ca * kv);
}

__device__ __forceinline__ const double *stream_x(const RowArgs<double> &a, int) { return a.fn; }
__device__ __forceinline__ const double *stream_y(const RowArgs<double> &a) { return a.f1; }
__device__ __forceinline__ const double *stream_z(const RowArgs<double> &a) { return a.f2; }
__device__ __forceinline__ const float *stream_x(const RowArgs<float> &a, int mode) {
  return mode == 1 ? a.fs : a.fn;
}
__device__ __forceinline__ const float *stream_y(const RowArgs<float> &a) { return a.acc; }
__device__ __forceinline__ const float *stream_z(const RowArgs<float> &) { return nullptr; }
__device__ __forceinline__ const float *rate_ref(const RowArgs<float> &a) { return a.rref; }
__device__ __forceinline__ const double *rate_ref(const RowArgs<double> &) { return nullptr; }
__device__ __forceinline__ const double *moments_ref(const RowArgs<float> &a) { return a.mref; }
__device__ __forceinline__ const double *moments_ref(const RowArgs<double> &) { return nullptr; }

// Column sums of the outputs a lane writes: value j of its accesses stays on
// one node, so 1, e_x and e_y times the outputs add up per value.
template <typename T>
struct ColumnSums {
  double s[3][16 / sizeof(T)];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int j = 0; j < (int)(16 / sizeof(T)); ++j) s[c][j] = 0.0;
  }
  __device__ __forceinline__ void add(int j, double o, double ex, double ey) {
    s[0][j] += o;
    s[1][j] += ex * o;
    s[2][j] += ey * o;
  }
};

// v + its values 32 (or 16) lanes away, for two values at a time: lanes 0..31
// (the even rows of 16 lanes) of the result hold a's sums, the others b's.
template <bool HALF>
__device__ __forceinline__ double fold_pair(double a, double b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (HALF) {
      const auto r = __builtin_amdgcn_permlane32_swap(x[i], y[i], false, false);
      x[i] = r[0];
      y[i] = r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(x[i], y[i], false, false);
      x[i] = r[0];
      y[i] = r[1];
    }
  }
  return __builtin_bit_cast(double, x) + __builtin_bit_cast(double, y);
}
// v + its value M lanes away in the row of 16 (rotation).
template <int M>
__device__ __forceinline__ double fold_row(double v) {
  typedef int i2 __attribute__((ext_vector_type(2)));
  const i2 x = __builtin_bit_cast(i2, v);
  i2 y;
#pragma unroll
  for (int i = 0; i < 2; ++i) y[i] = __builtin_amdgcn_update_dpp(0, x[i], 0x120 + M, 0xf, 0xf, false);
  return v + __builtin_bit_cast(double, y);
}

// A wavefront's sums of its lanes' columns over the access groups, in a fixed
// order, into red[parts][3][NP] (parts: row_sum_parts, summed by the reader);
// buf: the wavefront's tile.  Even node counts: the lanes of a column are a
// power of two apart and the sums fold across them in registers, two values at
// a time.  Odd ones go through LDS.
template <int P, typename T>
__device__ __forceinline__ void reduce_columns(const ColumnSums<T> &cs, int lane, double *buf, double *red) {
  using Sh = RowShape<P, T>;
  constexpr int NP = Sh::NP, VW = Sh::VW;
  if constexpr (Sh::PR == 1) {
    constexpr int N = 3 * VW, N2 = N / 2, N4 = (N2 + 1) / 2;
    double w[N2], u[N4];
#pragma unroll
    for (int i = 0; i < N2; ++i)
      w[i] = fold_pair<true>(cs.s[(2 * i) / VW][(2 * i) % VW], cs.s[(2 * i + 1) / VW][(2 * i + 1) % VW]);
#pragma unroll
    for (int i = 0; i < N4; ++i) {
      u[i] = fold_pair<false>(w[2 * i], w[2 * i + 1 < N2 ? 2 * i + 1 : 2 * i]);
      if (Sh::RA <= 8) u[i] = fold_row<8>(u[i]);
      if (Sh::RA <= 4) u[i] = fold_row<4>(u[i]);
      if (Sh::RA <= 2) u[i] = fold_row<2>(u[i]);
      if (Sh::RA <= 1) u[i] = fold_row<1>(u[i]);
    }
    const int row = lane >> 4, col = lane & 15;
    if (col < Sh::RA) {
#pragma unroll
      for (int i = 0; i < N4; ++i) {
        const int wi = 2 * i + (row & 1), vi = 2 * wi + (row >> 1);
        if (wi < N2) red[(vi / VW) * NP + VW * col + vi % VW] = u[i];
      }
    }
  } else {
    constexpr int L = Sh::G * Sh::RA, terms = Sh::G * Sh::PR, parts = row_sum_parts(NP, sizeof(T));
    constexpr bool ALL = row_sums_at_once(NP, sizeof(T));
    constexpr int O = ALL ? 3 * NP : NP;  // sums per round
    constexpr int each = (terms + parts - 1) / parts;
#pragma unroll
    for (int c0 = 0; c0 < 3; c0 += ALL ? 3 : 1) {
      wave_sync();
      if (lane < L) {
#pragma unroll
        for (int c = c0; c < (ALL ? 3 : c0 + 1); ++c)
#pragma unroll
          for (int j = 0; j < VW; ++j) buf[((c - c0) * L + lane) * VW + j] = cs.s[c][j];
      }
      wave_sync();
      for (int t = lane; t < O * parts; t += 64) {
        const int h = t / O, o = t - h * O, c = o / NP, n = o - c * NP;
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < each; ++i)
          if (h * each + i < terms) v += buf[c * L * VW + (h * each + i) * NP + n];
        red[h * 3 * NP + c0 * NP + o] = v;
      }
    }
  }
}

// The wall sums (outgoing normal speed times the state at the face nodes of
// each wall) of the rows lo..hi-1 of a tile; lane: face node m of face fc, rows
// h, h + H, ...
template <int P, typename T, typename A>
__device__ __forceinline__ double wall_sum(const A &a, const T *tile, int lo, int hi, int q0, int lane,
                                           const int (&nbr)[4]) {
  using Sh = RowShape<P, T>;
  constexpr int N1 = Sh::N1, F = 4 * N1, H = 64 / F;
  const int h = lane / F, fm = lane - h * F, fc = fm / N1, m = fm - fc * N1;
  const int node = fc == 0 ? m : fc == 1 ? m * N1 + P : fc == 2 ? P * N1 + m : m * N1;
  const bool on = h < H && (fc == 0 ? nbr[0] : fc == 1 ? nbr[1] : fc == 2 ? nbr[2] : nbr[3]) < 0;
  double s = 0.0;
  if (on) {
    const double *e = a.vel + (fc & 1 ? 0 : a.Q);
    const double sg = (fc == 1 || fc == 2) ? 1.0 : -1.0;
#pragma unroll 4
    for (int r = lo + h; r < hi; r += H) {
      const double en = sg * e[q0 + r];
      s += (en > 0.0 ? en : 0.0) * (double)tile[Sh::at(r, node)];
    }
  }
  return s;
}

// Loads of a wavefront's rows [r0, r0 + 64) counted from `base` (16-byte
// aligned) into registers, and from there into the tile.  Beyond nrows the last
// access is repeated (those rows are never read): with a branch per access
// instead, the sums of p = 3 took 214 registers, now 67, and problems with
// ragged wavefronts were 1 to 2% slower.
template <int P, typename T, typename V, int N>
__device__ __forceinline__ void tile_load(V (&v)[N], const T *base, int nrows, int lane) {
  using Sh = RowShape<P, T>;
  const int nacc = (nrows * Sh::NP + Sh::VW - 1) / Sh::VW;
#pragma unroll
  for (int u = 0; u < Sh::NLD; ++u) {
    const int c = min(lane + 64 * u, nacc - 1);
    v[u] = ld_stream<false, V>(base, 16u * c);
  }
}
template <int P, typename T, typename V, int N>
__device__ __forceinline__ void tile_store(const V (&v)[N], T *tile, int lane) {
  using Sh = RowShape<P, T>;
  constexpr int most = 64 * Sh::NP / Sh::VW;
#pragma unroll
  for (int u = 0; u < Sh::NLD; ++u) {
    const int c = lane + 64 * u;
    if (64 * u + 63 >= most && c >= most) continue;
    if constexpr (Sh::LIN) {
      *reinterpret_cast<V *>(tile + Sh::VW * c) = v[u];
    } else {
      constexpr int CPR = Sh::NP / Sh::VW > 0 ? Sh::NP / Sh::VW : 1;  // accesses per row
      const int r = c / CPR, w = c - r * CPR;
      *reinterpret_cast<V *>(tile + Sh::at(r, Sh::VW * w)) = v[u];
    }
  }
}

// Accesses in flight per lane and stream in the update pass.
template <int P, typename T, int MODE, bool REF>
constexpr int update_batch() {
  constexpr int NIT = RowShape<P, T>::NIT;
  constexpr int most = sizeof(T) == 8 && P == 2 ? 5 : 4;
  return NIT < most ? NIT : (NIT + (NIT + most - 1) / most - 1) / ((NIT + most - 1) / most);
}

// The operands of a batch of the update: U accesses per lane from pass it0.
// Loads are unconditional (accesses past the last row repeat it) so that all of
// them are in flight together.
template <int P, typename T, int MODE, bool REF>
struct Operands {
  using Sh = RowShape<P, T>;
  using St = Streams<T, MODE>;
  using V = typename VecOf<T>::type;
  static constexpr int U = update_batch<P, T, MODE, REF>();
  V x[U], y[U], z[U], r[U];
  template <bool NT, typename A>
  __device__ __forceinline__ void load(const A &a, ptrdiff_t off, int it0, int rlast, int g, int w) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int rb = min(Sh::PR * (g + Sh::G * (it0 + u)), rlast);
      const unsigned at = (unsigned)(rb * Sh::NP + Sh::VW * w) * (unsigned)sizeof(T);
      if constexpr (REF) r[u] = ld_stream<NT, V>(rate_ref(a) + off, at);
      if constexpr (St::X) x[u] = ld_stream<NT, V>(stream_x(a, MODE) + off, at);
      if constexpr (St::Y) y[u] = ld_stream<NT, V>(stream_y(a) + off, at);
      if constexpr (St::Z) z[u] = ld_stream<NT, V>(stream_z(a) + off, at);
    }
  }
};

// The update pass over a wavefront's rows lo..hi-1 (tile: the row phase's
// results; off: offset of the tile's first row in the states), and with SUM the
// column sums of its outputs, with keep the outputs back into the tile.  ev:
// e_x, e_y of the tile's rows.  (Its operands loaded before the rows are
// evaluated, where registers allow it, measured 2 to 15% slower.)  WHOLE: 64
// rows of this element; else rows of another one (the lead, or what the last
// access holds beyond this element) are neither stored nor summed.
template <int P, typename T, int MODE, bool REF, bool NT, bool SUM, bool WHOLE, typename A>
__device__ __forceinline__ void rows_update_pass(const A &a, T *tile, const d2 *ev, ptrdiff_t off, int lo, int hi,
                                                 int lane, bool keep, ColumnSums<T> &cs) {
  using Sh = RowShape<P, T>;
  using St = Streams<T, MODE>;
  using V = typename VecOf<T>::type;
  constexpr int NP = Sh::NP, VW = Sh::VW, PR = Sh::PR, NIT = Sh::NIT;
  constexpr int U = Operands<P, T, MODE, REF>::U;
  T *accr = a.acc + off, *outr = a.out + off;
  const int g = lane / Sh::RA, w = lane - g * Sh::RA;
  if (Sh::G * Sh::RA < 64 && g >= Sh::G) return;  // lanes beyond the last group
  const int r1 = (VW * w) / NP, r2 = (VW * w + VW - 1) / NP;  // first and last row of an access, within the period
  const int cross = r2 > r1 ? r2 * NP - VW * w : VW;           // first value of the last row
  const int rlast = WHOLE ? 64 - PR : (hi - 1) / PR * PR;      // last period with a row
  const int nit = WHOLE ? NIT : (hi + Sh::RPI - 1) / Sh::RPI;
#pragma unroll 1
  for (int it0 = 0; it0 < nit; it0 += U) {
    Operands<P, T, MODE, REF> op;
    op.template load<NT>(a, off, it0, rlast, g, w);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (WHOLE && NIT % U != 0 && it0 + u >= NIT) continue;
      const bool clamp = !WHOLE || (Sh::RPI * NIT > 64 && (it0 + u + 1) * Sh::RPI > 64);
      const int rb0 = PR * (g + Sh::G * (it0 + u)), rb = clamp ? min(rb0, rlast) : rb0;
      const unsigned pos = (unsigned)(rb * NP + VW * w);
      T *t = Sh::LIN ? tile + pos : tile + Sh::at(rb, VW * w);
      const V kv = *reinterpret_cast<const V *>(t);
      V o, an;
#pragma unroll
      for (int j = 0; j < VW; ++j) {
        T k = kv[j], aj = 0, xj = 0, yj = 0, zj = 0;
        if constexpr (REF) k += op.r[u][j];
        if constexpr (St::X) xj = op.x[u][j];
        if constexpr (St::Y) yj = op.y[u][j];
        if constexpr (St::Z) zj = op.z[u][j];
        o[j] = update_value<MODE>(k, xj, yj, zj, a.c_acc, a.c_out, aj);
        an[j] = aj;
      }
      const bool here = !clamp || rb0 <= rlast;
      const bool first = WHOLE ? here : here && rb + r1 >= lo && rb + r1 < hi;
      const bool last = WHOLE ? here : here && rb + r2 >= lo && rb + r2 < hi;
      if (MODE == kRateSums) {  // (nothing is stored)
      } else if (first && last) {
        st_stream<NT, V>(outr, pos * (unsigned)sizeof(T), o);
        if constexpr (St::ACC) st_stream<NT, V>(accr, pos * (unsigned)sizeof(T), an);
      } else if (!WHOLE && PR > 1 && (first || last)) {
#pragma unroll
        for (int j = 0; j < VW; ++j)
          if (j < cross ? first : last) {
            outr[pos + j] = o[j];
            if constexpr (St::ACC) accr[pos + j] = an[j];
          }
      }
      if constexpr (SUM) {
        const d2 e1 = ev[rb + r1];
        d2 e2 = e1;
        if constexpr (PR > 1) e2 = ev[rb + r2];
#pragma unroll
        for (int j = 0; j < VW; ++j) {
          const bool in1 = PR == 1 || j == 0 || (j < VW - 1 && j < cross);
          const bool counts = in1 ? first : last;
          const double oj = counts ? (double)o[j] : 0.0;
          cs.add(j, oj, in1 ? e1[0] : e2[0], in1 ? e1[1] : e2[1]);
        }
        if (keep && here) *reinterpret_cast<V *>(t) = o;
      }
    }
  }
}

template <int P, typename T, int MODE, bool REF, bool SUM, typename A>
__device__ __forceinline__ void rows_update(const A &a, T *tile, const d2 *ev, ptrdiff_t off, int lo, int hi,
                                            int lane, bool keep, ColumnSums<T> &cs) {
  if (lo != 0 || hi != 64)
    rows_update_pass<P, T, MODE, REF, false, SUM, false>(a, tile, ev, off, lo, hi, lane, keep, cs);
  else if (a.stream_nt)
    rows_update_pass<P, T, MODE, REF, true, SUM, true>(a, tile, ev, off, 0, 64, lane, keep, cs);
  else
    rows_update_pass<P, T, MODE, REF, false, SUM, true>(a, tile, ev, off, 0, 64, lane, keep, cs);
}

// What a lane needs of its row beside the values: the velocity and the exterior
// traces of its two inflow faces.  Loaded before
// the tile is in LDS, so that the traces travel with it.
template <int P, typename T>
struct RowIn {
  T cx, cy, wq;
  double cxd, cyd, wqd;
  int nbx, nby;
  T px[P + 1], py[P + 1];
};

template <int P, typename T, typename A>
__device__ __forceinline__ void row_velocity(const A &a, int q, RowIn<P, T> &in) {
  in.cxd = a.vel[q];
  in.cyd = a.vel[a.Q + q];
  in.wqd = a.vel[2 * a.Q + q];
}

// Velocity q of element k; nbl .. nbt: its neighbours (-1: wall, whose trace
// row_walls forms; some row of its own is loaded).
template <int P, typename T, typename A>
__device__ __forceinline__ void row_traces_load(const A &a, int k, int q, int nbl, int nbr, int nbb, int nbt,
                                                RowIn<P, T> &in) {
  using Sh = RowShape<P, T>;
  constexpr int N1 = Sh::N1, NP = Sh::NP;
  const T cx = in.cx = (T)in.cxd, cy = in.cy = (T)in.cyd;
  in.wq = (T)in.wqd;
  const int nbx = in.nbx = cx > 0 ? nbl : nbr, nby = in.nby = cy > 0 ? nbb : nbt;
  const T *sx = a.fs + ((size_t)(nbx >= 0 ? nbx : k) * a.Q + q) * NP + (cx > 0 ? P : 0);
  const T *sy = a.fs + ((size_t)(nby >= 0 ? nby : k) * a.Q + q) * NP + (cy > 0 ? N1 * P : 0);
#pragma unroll
  for (int m = 0; m < N1; ++m) in.px[m] = sx[N1 * m];
  if constexpr (N1 * sizeof(T) % 16 == 0) {
    using V = typename VecOf<T>::type;
#pragma unroll
    for (int m = 0; m < N1; m += Sh::VW) {
      const V v = *reinterpret_cast<const V *>(sy + m);
#pragma unroll
      for (int j = 0; j < Sh::VW; ++j) in.py[m + j] = v[j];
    }
  } else {
#pragma unroll
    for (int m = 0; m < N1; ++m) in.py[m] = sy[m];
  }
}

// Traces at a wall: its diffuse reflection rho_w f^eq(1, u_b) (FP32 storage: as
// a deviation from w rho_ref); rwe: the element's wall densities.
template <int P, typename T, bool REF, typename A>
__device__ __forceinline__ void row_walls(const A &a, int q, const double *rwe, RowIn<P, T> &in) {
  constexpr int N1 = P + 1;
  double wrr = 0.0;
  if constexpr (sizeof(T) == 4 && !REF) wrr = in.wqd * a.rho_ref;
  if (in.nbx < 0) {
    const int fc = in.cx > 0 ? 3 : 1;
    const double gb = a.feqb[fc * a.Q + q];
#pragma unroll
    for (int m = 0; m < N1; ++m) in.px[m] = (T)(rwe[fc * N1 + m] * gb - wrr);
  }
  if (in.nby < 0) {
    const int fc = in.cy > 0 ? 0 : 2;
    const double gb = a.feqb[fc * a.Q + q];
#pragma unroll
    for (int m = 0; m < N1; ++m) in.py[m] = (T)(rwe[fc * N1 + m] * gb - wrr);
  }
}

// Row phase: L(f) of the tile's row r (or what its stage makes of it) over the
// row's place in the tile; mm: the element's node factors.
template <int P, typename T, int MODE, bool REF, typename A>
__device__ __forceinline__ void row_phase(const A &a, T *tile, int r, const RowIn<P, T> &in, const T *mm) {
  using Sh = RowShape<P, T>;
  constexpr int NP = Sh::NP;
  T f[NP], kk[NP];
  if constexpr (NP % Sh::VW == 0) {
    using V = typename VecOf<T>::type;
#pragma unroll
    for (int c = 0; c < NP; c += Sh::VW) {
      const V v = *reinterpret_cast<const V *>(tile + Sh::at(r, c));
#pragma unroll
      for (int j = 0; j < Sh::VW; ++j) f[c + j] = v[j];
    }
  } else {
#pragma unroll
    for (int c = 0; c < NP; ++c) f[c] = tile[r * Sh::S + c];
  }
  row_transport<P>(a, f, in.cx, in.cy, in.px, in.py, kk);
  row_collide<P, REF>(a, mm, in.cx, in.cy, in.wq, f, kk);
  row_result<MODE>(a, f, kk);
  if constexpr (NP % Sh::VW == 0) {
    using V = typename VecOf<T>::type;
#pragma unroll
    for (int c = 0; c < NP; c += Sh::VW) {
      V v;
#pragma unroll
      for (int j = 0; j < Sh::VW; ++j) v[j] = kk[c + j];
      *reinterpret_cast<V *>(tile + Sh::at(r, c)) = v;
    }
  } else {
#pragma unroll
    for (int c = 0; c < NP; ++c) tile[r * Sh::S + c] = kk[c];
  }
}

// ---- handed-over moments: one element per work-group --------------------------

// max that keeps NaN
__device__ __forceinline__ double nan_max(double a, double b) { return (b > a || b != b) ? b : a; }

// The wavefront's largest m into *result, the bit pattern of a non-negative
// double (which orders as the values do, NaN above all).  Most wavefronts find
// a larger value there already and leave it.
__device__ __forceinline__ void max_out(double m, unsigned long long *result) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = nan_max(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(fabs(m));
    if (bits > __hip_atomic_load(result, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(result, bits);
  }
}

// The work-group's sums from its wavefronts' columns, in a fixed order; red: LDS
// of their own for the wavefronts' sums (the wall sums pass through the tiles).
// RATES: of one velocity tile, the sums are the node's moment rates and their
// largest goes to *result.
template <int P, typename T, bool RATES = false>
__device__ __forceinline__ void rows_sums_out(const ColumnSums<T> &cs, double ws, bool wall, int wave, int lane,
                                              int nw, bool on, const int (&nbr)[4], char *lds, double *red,
                                              double *po, double scale = 0.0,
                                              unsigned long long *result = nullptr) {
  using Sh = RowShape<P, T>;
  constexpr int N1 = Sh::N1, NP = Sh::NP, F = 4 * N1, H = 64 / F, parts = row_sum_parts(NP, sizeof(T));
  constexpr int WB = row_wave_bytes(NP, sizeof(T)) + 64 * 16;
  if (on) {
    double *buf = reinterpret_cast<double *>(lds + wave * WB);
    reduce_columns<P, T>(cs, lane, buf, red + wave * parts * 3 * NP);
    if (wall) {
      wave_sync();
      buf[lane] = ws;
    }
  }
  __syncthreads();
  if (!on) return;
  const int tid = 64 * wave + lane;
  double m = 0.0;
  for (int t = tid; t < 3 * NP; t += 64 * nw) {
    double s = 0.0;
    for (int wv = 0; wv < nw * parts; ++wv) s += red[wv * 3 * NP + t];
    if (RATES && result) m = nan_max(m, fabs(s) * scale);
    else po[t] = s;
  }
  if (RATES) {
    if (result && 64 * wave < 3 * NP) max_out(m, result);
    return;
  }
  if (wall && tid < F) {
    const int fc = tid / N1, m = tid - fc * N1;
    if ((fc == 0 ? nbr[0] : fc == 1 ? nbr[1] : fc == 2 ? nbr[2] : nbr[3]) < 0) {
      double s = 0.0;
      for (int wv = 0; wv < nw; ++wv) {
        const double *buf = reinterpret_cast<const double *>(lds + wv * WB);
#pragma unroll
        for (int h = 0; h < H; ++h) s += buf[h * F + tid];
      }
      const int node = fc == 0 ? m : fc == 1 ? m * N1 + P : fc == 2 ? P * N1 + m : m * N1;
      po[(3 + fc) * NP + node] = s;
    }
  }
}

// Element k, velocity tile vt, by nw wavefronts of a work-group; wave: which of
// them; on: whether there is such an element (the barriers are passed anyway).
template <int P, typename T, int MODE, bool REF, typename A>
__device__ __forceinline__ void rows_element(const A &a, int k, int vt, int wave, bool on, char *lds) {
  using Sh = RowShape<P, T>;
  using V = typename VecOf<T>::type;
  constexpr int N1 = Sh::N1, NP = Sh::NP, MS = node_values<T, REF>();
  constexpr int TB = row_wave_bytes(NP, sizeof(T)), WB = TB + 64 * 16;
  const int lane = threadIdx.x & 63, tid = 64 * wave + lane;
  const int nw = a.nw, Q = a.Q;
  T *tile = reinterpret_cast<T *>(lds + wave * WB);
  d2 *ev = reinterpret_cast<d2 *>(lds + wave * WB + TB);
  char *shared = lds + nw * WB;
  T *mom = reinterpret_cast<T *>(shared);
  double *rw = reinterpret_cast<double *>(shared + (NP * MS * sizeof(T) + 15) / 16 * 16);
  double *red = rw + 4 * N1;
  const int ey = quotient(k, a.dnx), ex = k - ey * a.nx;
  const int nbr[4] = {row_neighbour(ex, ey, k, 0, a), row_neighbour(ex, ey, k, 1, a),
                      row_neighbour(ex, ey, k, 2, a), row_neighbour(ex, ey, k, 3, a)};
  const bool wall = nbr[0] < 0 || nbr[1] < 0 || nbr[2] < 0 || nbr[3] < 0;
  const size_t row0 = (size_t)k * Q;
  const int lead = (int)(row0 % Sh::PR);
  const ptrdiff_t base = (ptrdiff_t)(row0 - lead) * NP;
  const int vrows = Q + lead;  // rows counted from the aligned one
  const int nch = (vrows + 63) >> 6;

  const int c = vt * nw + wave;  // this wavefront's rows: 64 from 64 c
  const bool work = on && c < nch;
  const int lo = max(0, lead - 64 * c), hi = min(64, vrows - 64 * c), q0 = 64 * c - lead;
  const int q = min(max(q0 + lane, 0), Q - 1);

  // loads, all issued before any is waited for: the row's velocity, the
  // element's moment sums, the rows, and (their addresses need the velocity's
  // signs) the traces
  RowIn<P, T> in;
  if (work) row_velocity<P, T>(a, q, in);
  double sm[3] = {0.0, 0.0, 0.0}, sw[4] = {0.0, 0.0, 0.0, 0.0}, ref[3] = {0.0, 0.0, 0.0};
  // At p = 4, where an element usually takes several velocity tiles, the tiles'
  // sums are all in flight with the rows (one wait per tile before the first
  // wavefront's rows otherwise: 128x128 elements, 576 velocities, a step 5.06 ->
  // 4.96 ms in FP64, 3.41 -> 3.37 in FP32; at p = 2 it costs 1%).
  constexpr bool TOGETHER = P == 4;
  double pv[TOGETHER ? kMaxPartialTiles : 1][3];
  const bool loads_moments = on && tid < NP;
  if (loads_moments) {
    if constexpr (TOGETHER) {
#pragma unroll
      for (int t = 0; t < kMaxPartialTiles; ++t) {
        if (t >= a.nt) break;
        const double *pp = a.pin + ((size_t)t * a.K + k) * 7 * NP + tid;
#pragma unroll
        for (int c = 0; c < 3; ++c) pv[t][c] = pp[c * NP];
      }
    }
    if (!TOGETHER || wall) {
#pragma unroll 1
      for (int t = 0; t < a.nt; ++t) {
        const double *pp = a.pin + ((size_t)t * a.K + k) * 7 * NP + tid;
        if constexpr (!TOGETHER) {
#pragma unroll
          for (int c = 0; c < 3; ++c) sm[c] += pp[c * NP];
        }
        if (wall) {
#pragma unroll
          for (int c = 0; c < 4; ++c) sw[c] += pp[(3 + c) * NP];
        }
      }
    }
    if constexpr (REF) {
      const size_t KN = (size_t)a.K * NP, node = (size_t)k * NP + tid;
#pragma unroll
      for (int c = 0; c < 3; ++c) ref[c] = moments_ref(a)[c * KN + node];
    }
  }
  V v[Sh::NLD];
  const ptrdiff_t off = base + (ptrdiff_t)c * 64 * NP;
  if (work) {
    tile_load<P, T>(v, a.fs + off, hi, lane);
    row_traces_load<P, T>(a, k, q, nbr[3], nbr[1], nbr[0], nbr[2], in);
  }
  if (loads_moments) {
    if constexpr (TOGETHER) {
#pragma unroll
      for (int t = 0; t < kMaxPartialTiles; ++t) {
        if (t >= a.nt) break;
#pragma unroll
        for (int c = 0; c < 3; ++c) sm[c] += pv[t][c];
      }
    }
    node_factors_t<REF>(a, sm, ref, mom + tid * MS);
    if (wall) {
      const int i = tid % N1, j = tid / N1;
      const bool on[4] = {nbr[0] < 0 && j == 0, nbr[1] < 0 && i == P, nbr[2] < 0 && j == P, nbr[3] < 0 && i == 0};
      const int fm[4] = {i, j, i, j};
#pragma unroll
      for (int fc = 0; fc < 4; ++fc)
        if (on[fc]) rw[fc * N1 + fm[fc]] = (sw[fc] + wall_const<REF>(a, fc)) * a.wall_den_inv[fc];
    }
  }
  if (work) {
    tile_store<P, T>(v, tile, lane);
    ev[lane] = d2{in.cxd, in.cyd};
  }
  __syncthreads();

  ColumnSums<T> cs;
  cs.clear();
  double ws = 0.0;
  if (work) {
    if (wall) row_walls<P, T, REF>(a, q, rw, in);
    if (lane >= lo && lane < hi) row_phase<P, T, MODE, REF>(a, tile, lane, in, mom);
    wave_sync();
    constexpr bool SUM = row_sums_mode(MODE), WALLS = SUM && MODE != kRateSums;
    rows_update<P, T, MODE, REF, SUM>(a, tile, ev, off, lo, hi, lane, WALLS && wall, cs);
    if (WALLS && wall) {
      wave_sync();
      ws = wall_sum<P, T>(a, tile, lo, hi, q0, lane, nbr);
    }
  }
  if constexpr (!row_sums_mode(MODE)) return;
  double *po = a.pout + ((size_t)vt * a.K + k) * 7 * NP;
  if constexpr (MODE == kRateSums)
    rows_sums_out<P, T, true>(cs, ws, false, wave, lane, nw, on, nbr, lds, red, po, a.resid_scale,
                              a.nt == 1 ? a.result : nullptr);
  else
    rows_sums_out<P, T>(cs, ws, wall, wave, lane, nw, on, nbr, lds, red, po);
}

// The same sums of a state as it is (after it was set from outside a step), by
// the same lanes in the same order, so that a state read out and set again
// continues bit for bit.  Bound by the one read; summed by the update's pass
// with its velocities in LDS (read from memory in the loop, 2.4 million FP64
// values took 15.4 us, now 6.7).
template <int P, typename T, typename A>
__device__ __forceinline__ void rows_state_sums(const A &a, int k, int vt, char *lds) {
  using Sh = RowShape<P, T>;
  using V = typename VecOf<T>::type;
  constexpr int NP = Sh::NP, PR = Sh::PR;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int nw = a.nw, Q = a.Q;
  constexpr int TB = row_wave_bytes(NP, sizeof(T)), WB = TB + 64 * 16;
  T *tile = reinterpret_cast<T *>(lds + wave * WB);
  d2 *ev = reinterpret_cast<d2 *>(lds + wave * WB + TB);
  double *red = reinterpret_cast<double *>(lds + nw * WB);
  const int ey = quotient(k, a.dnx), ex = k - ey * a.nx;
  const int nbr[4] = {row_neighbour(ex, ey, k, 0, a), row_neighbour(ex, ey, k, 1, a),
                      row_neighbour(ex, ey, k, 2, a), row_neighbour(ex, ey, k, 3, a)};
  const bool wall = nbr[0] < 0 || nbr[1] < 0 || nbr[2] < 0 || nbr[3] < 0;
  const size_t row0 = (size_t)k * Q;
  const int lead = (int)(row0 % PR);
  const ptrdiff_t base = (ptrdiff_t)(row0 - lead) * NP;
  const int vrows = Q + lead, nch = (vrows + 63) >> 6;
  ColumnSums<T> cs;
  cs.clear();
  double ws = 0.0;
  const int c = vt * nw + wave;
  if (c < nch) {
    const int lo = max(0, lead - 64 * c), hi = min(64, vrows - 64 * c), q0 = 64 * c - lead;
    V v[Sh::NLD];
    tile_load<P, T>(v, a.fs + base + (ptrdiff_t)c * 64 * NP, hi, lane);
    const int q = min(max(q0 + lane, 0), Q - 1);
    ev[lane] = d2{a.vel[q], a.vel[Q + q]};
    wave_sync();
    tile_store<P, T>(v, tile, lane);
    wave_sync();
    rows_update<P, T, kRateSums, false, true>(a, tile, ev, base + (ptrdiff_t)c * 64 * NP, lo, hi, lane, false, cs);
    if (wall) ws += wall_sum<P, T>(a, tile, lo, hi, q0, lane, nbr);
  }
  rows_sums_out<P, T>(cs, ws, wall, wave, lane, nw, true, nbr, lds, red,
                      a.pout + ((size_t)vt * a.K + k) * 7 * NP);
}

// ---- moments in the wavefront: a.ew whole elements per wavefront ---------------

// w: which run of a.ew elements.
template <int P, typename T, int MODE, bool REF, typename A>
__device__ __forceinline__ void rows_wave(const A &a, int w, char *lds) {
  using Sh = RowShape<P, T>;
  using V = typename VecOf<T>::type;
  constexpr int N1 = Sh::N1, NP = Sh::NP, MS = node_values<T, REF>();
  constexpr int ES = row_node_stride(NP, sizeof(T), REF);
  const int lane = threadIdx.x & 63, Q = a.Q, k0 = w * a.ew;
  const int Eb = min(a.ew, a.K - k0);
  T *tile = reinterpret_cast<T *>(lds);
  constexpr int TB = row_wave_bytes(NP, sizeof(T));
  d2 *ev = reinterpret_cast<d2 *>(lds + TB);  // e_x, e_y of the rows
  T *mom = reinterpret_cast<T *>(lds + TB + 64 * 16);
  double *rw = reinterpret_cast<double *>(lds + TB + 64 * 16 + (a.ew * ES * (int)sizeof(T) + 15) / 16 * 16);
  const size_t row0 = (size_t)k0 * Q;
  const int lead = (int)(row0 % Sh::PR);
  const ptrdiff_t base = (ptrdiff_t)(row0 - lead) * NP;
  const int hi = lead + Eb * Q;  // at most 64
  // this lane's row
  const int r = max(min(lane, hi - 1) - lead, 0), er = (r >= Q) + (r >= 2 * Q) + (r >= 3 * Q), q = r - er * Q,
            kr = k0 + er;
  const int ey0 = quotient(k0, a.dnx), ex0 = k0 - ey0 * a.nx;
  int exr, eyr;
  step_place(ex0, ey0, er, a, exr, eyr);
  RowIn<P, T> in;
  row_velocity<P, T>(a, q, in);
  V v[Sh::NLD];
  tile_load<P, T>(v, a.fs + base, hi, lane);
  row_traces_load<P, T>(a, kr, q, row_neighbour(exr, eyr, kr, 3, a), row_neighbour(exr, eyr, kr, 1, a),
                        row_neighbour(exr, eyr, kr, 0, a), row_neighbour(exr, eyr, kr, 2, a), in);
  tile_store<P, T>(v, tile, lane);
  ev[lane] = d2{in.cxd, in.cyd};
  wave_sync();

  // node moments: lane (part h, element e, node n) sums velocities h, h + H,
  // ... from the tile; the parts of a node are `per` lanes apart
  const int H = min(4, max(1, 64 / (NP * a.ew))), per = 64 / H;
  for (int t0 = 0; t0 < Eb * NP; t0 += per) {
    const int h = lane / per, t = t0 + lane - h * per;
    const int e = t / NP, n = t - e * NP, i = n % N1, j = n / N1;
    const bool in = h < H && t < Eb * NP;
    double sm[3] = {0.0, 0.0, 0.0}, sw[4] = {0.0, 0.0, 0.0, 0.0}, ref[3] = {0.0, 0.0, 0.0};
    bool on[4] = {false, false, false, false};
    if constexpr (REF) {
      if (in && h == 0) {
        const size_t KN = (size_t)a.K * NP, node = (size_t)(k0 + e) * NP + n;
#pragma unroll
        for (int c = 0; c < 3; ++c) ref[c] = moments_ref(a)[c * KN + node];
      }
    }
    if (in && a.wall_mask) {
      const int k = k0 + e;
      int ex, ey;
      step_place(ex0, ey0, e, a, ex, ey);
      on[0] = j == 0 && row_neighbour(ex, ey, k, 0, a) < 0;
      on[1] = i == P && row_neighbour(ex, ey, k, 1, a) < 0;
      on[2] = j == P && row_neighbour(ex, ey, k, 2, a) < 0;
      on[3] = i == 0 && row_neighbour(ex, ey, k, 3, a) < 0;
    }
    const bool walls = __any(on[0] || on[1] || on[2] || on[3]);
    if (in) {
      const int rq = lead + e * Q;
#pragma unroll 4
      for (int q = h; q < Q; q += H) {
        const double o = (double)tile[Sh::at(rq + q, n)], cx = ev[lead + q][0], cy = ev[lead + q][1];
        sm[0] += o;
        sm[1] += cx * o;
        sm[2] += cy * o;
        if (walls) {
          sw[0] += (cy < 0.0 ? -cy : 0.0) * o;
          sw[1] += (cx > 0.0 ? cx : 0.0) * o;
          sw[2] += (cy > 0.0 ? cy : 0.0) * o;
          sw[3] += (cx < 0.0 ? -cx : 0.0) * o;
        }
      }
    }
    for (int s = 1; s < H; ++s) {
      const int from = (lane + s * per) & 63;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double o = __shfl(sm[c], from);
        if (h == 0) sm[c] += o;
      }
      if (walls) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double o = __shfl(sw[c], from);
          if (h == 0) sw[c] += o;
        }
      }
    }
    if (in && h == 0) {
      node_factors_t<REF>(a, sm, ref, mom + e * ES + n * MS);
      const int fm[4] = {i, j, i, j};
#pragma unroll
      for (int fc = 0; fc < 4; ++fc)
        if (on[fc]) rw[(e * 4 + fc) * N1 + fm[fc]] = (sw[fc] + wall_const<REF>(a, fc)) * a.wall_den_inv[fc];
    }
  }
  wave_sync();
  if (a.wall_mask) row_walls<P, T, REF>(a, q, rw + er * 4 * N1, in);
  if (lane >= lead && lane < hi) row_phase<P, T, MODE, REF>(a, tile, lane, in, mom + er * ES);
  wave_sync();
  if constexpr (MODE == kRateSums) {
    // the node's moment rates, by the lanes that summed its moments
    double m = 0.0;
    for (int t0 = 0; t0 < Eb * NP; t0 += per) {
      const int h = lane / per, t = t0 + lane - h * per;
      const int e = t / NP, n = t - e * NP;
      double sm[3] = {0.0, 0.0, 0.0};
      if (h < H && t < Eb * NP) {
        const int rq = lead + e * Q;
        for (int q = h; q < Q; q += H) {
          T k = tile[Sh::at(rq + q, n)];
          if constexpr (REF) k += rate_ref(a)[base + (ptrdiff_t)(rq + q) * NP + n];
          sm[0] += (double)k;
          sm[1] += ev[rq + q][0] * (double)k;
          sm[2] += ev[rq + q][1] * (double)k;
        }
      }
      for (int s = 1; s < H; ++s) {
        const int from = (lane + s * per) & 63;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double o = __shfl(sm[c], from);
          if (h == 0) sm[c] += o;
        }
      }
      if (h == 0 && t < Eb * NP)
#pragma unroll
        for (int c = 0; c < 3; ++c) m = nan_max(m, fabs(sm[c]) * a.resid_scale);
    }
    max_out(m, a.result);
    return;
  }
  ColumnSums<T> cs;  // (not summed here)
  rows_update<P, T, MODE, REF, false>(a, tile, nullptr, base, lead, hi, lane, false, cs);
}

// ---- kernels ---------------------------------------------------------------------

// The b-th work-group's place: the 8 XCDs take work-groups round-robin, so
// each gets a contiguous run, swept in strips 16 elements wide, so that the
// work-groups resident on one XCD cover a compact patch and find their
// neighbours' faces in its L2.
__device__ __forceinline__ int xcd_run(int b, int n) {
  const int per = n >> 3, rem = n & 7, x = b & 7;
  return x * per + (x < rem ? x : rem) + (b >> 3);
}
template <typename A>
__device__ __forceinline__ int strip_place(int t, const A &a) {
  const int W = a.strip_w;  // work-groups per strip (0: in mesh order)
  if (W == 0) return t;
  const int strip = quotient(t, a.dstrip), in = t - strip * (int)a.dstrip.d;
  const bool whole = strip < a.strips;  // (the last strip may be narrower)
  const int w = whole ? W : a.strip_last;
  const int row = whole ? quotient(in, a.dw) : quotient(in, a.dlast);
  return row * a.strip_row + strip * W + in - row * w;
}

constexpr int kKindElement = 1, kKindWave = 2, kKindSums = 3;
template <int KIND>
constexpr int row_threads() { return KIND == kKindWave ? 64 : 256; }

// Wavefronts per SIMD asked of the compiler: what fits without spilling a
// vector register; the build refuses scratch in these kernels.  A request that
// spilled once gave wrong rates.  Why is not known: in 69 instantiations compiled
// to spill, and not run, every reload reads what the lanes that are on there
// had stored.
template <int KIND, int P, typename T, int MODE>
constexpr int row_waves() {
  if (KIND == kKindSums) return 1;
  if (MODE == kRateSums && P == 4) return sizeof(T) == 8 && KIND == kKindWave ? 2 : 3;
  if (KIND == kKindWave) return sizeof(T) == 8 ? (P <= 2 ? 4 : P == 3 ? 3 : 2) : 4;
  if (sizeof(T) == 8) return P == 1 ? 6 : P == 2 ? 5 : P == 3 ? 4 : 3;
  return P == 1 ? 6 : P == 2 ? 5 : 4;
}

// (aimed at five, the FP32 kernels of p = 4 spill, their rate sums aimed at
// four, the FP64 rate sums of a batch aimed at three)
template <int KIND, int P, typename T, int MODE>
constexpr int row_waves_most() {
  return P < 4 ? 8 : MODE == kRateSums ? (sizeof(T) == 8 && KIND == kKindWave ? 2 : 3) : sizeof(T) == 4 ? 4 : 8;
}

template <int KIND, int P, typename T, int MODE, bool REF, typename A>
__device__ __forceinline__ void rows_body(const A &a, int b, int vt, char *lds) {
  if constexpr (KIND == kKindElement)
    rows_element<P, T, MODE, REF>(a, b, vt, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), true, lds);
  else if constexpr (KIND == kKindWave) rows_wave<P, T, MODE, REF>(a, b, lds);
  else rows_state_sums<P, T>(a, b, vt, lds);
}

template <int KIND, int P, typename T, int MODE, bool REF, typename A>
__global__ __launch_bounds__(row_threads<KIND>())
__attribute__((amdgpu_waves_per_eu(row_waves<KIND, P, T, MODE>(), row_waves_most<KIND, P, T, MODE>())))
void rows_kernel(const A a) {
  extern __shared__ char row_lds[];
  const int b = strip_place(xcd_run(blockIdx.x, a.nblk), a);
  rows_body<KIND, P, T, MODE, REF>(a, b, blockIdx.y, row_lds);
}

// One item of a batch: the at-th work-group of four wavefronts of the problem's
// plan (kind 1: as many elements and velocity tiles as they take; kind 2: four
// runs of elements).  Bound by how many wavefronts are in flight: a work-group
// of two wavefronts held a slot of four.  Eight problems of 16x16 to 28x28
// elements, p = 2 and 3, 16 to 100 velocities, per step: FP64 107 -> 83 us,
// FP32_REF 98 -> 78 us.
template <int P, typename T, int MODE, bool REF, typename A>
__device__ __forceinline__ void rows_item(const A &a, int at, char *lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a.kind == kKindElement) {
    const int nw = a.nw, per = nw == 2 ? 2 : 1, sub = nw == 2 ? wave >> 1 : 0;
    const int i = at * per + sub, w = wave - sub * nw;  // (of three wavefronts' elements the fourth sits out)
    const bool on = w < nw && i < a.nblk * a.nt;
    const int k = on ? quotient(i, a.dnt) : 0;
    rows_element<P, T, MODE, REF>(a, k, on ? i - k * a.nt : 0, w, on, lds + sub * a.lds);
  } else {
    const int w = 4 * at + wave;
    if (w < a.nblk)
      rows_wave<P, T, MODE, REF>(a, w, lds + wave * a.lds);
  }
}

// One work-group per item (problem, work-group of its plan), listed in the order
// the XCDs take them; the arguments come from a descriptor table in the constant
// address space (scalar loads).
template <int P, typename T, int MODE, bool REF, typename A>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(row_waves<kKindWave, P, T, MODE>(), row_waves_most<kKindWave, P, T, MODE>())))
void batch_rows_kernel(const A *descs, const int2 *items, int nitems) {
  extern __shared__ char row_lds[];
  const int2 it = items[blockIdx.x];
  const int inst = __builtin_amdgcn_readfirstlane(it.x), at = __builtin_amdgcn_readfirstlane(it.y);
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(4))) const A ConstArgs;
  const A a = ((ConstArgs *)descs)[inst];
#else
  const A a = descs[inst];  // host pass: the body is never run on the host
#endif
  rows_item<P, T, MODE, REF>(a, at, row_lds);
}

template <int KIND, int P, typename T, int MODE, bool REF, typename A>
hipError_t launch_one(const A &a, size_t lds, hipStream_t st) {
  constexpr int kind = KIND == kKindSums ? kKindElement : KIND;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void *)rows_kernel<KIND, P, T, MODE, REF, A>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int threads = kind == kKindElement ? 64 * a.nw : 64;
  const dim3 grid((unsigned)a.nblk, kind == kKindElement ? (unsigned)a.nt : 1u);
  hipLaunchKernelGGL((rows_kernel<KIND, P, T, MODE, REF, A>), grid, dim3(threads), lds, st, a);
  return hipGetLastError();
}

template <int P, typename T, int MODE, bool REF, typename A>
hipError_t launch_batch_one(const A *descs, const int2 *items, int nitems, size_t lds, hipStream_t st) {
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void *)batch_rows_kernel<P, T, MODE, REF, A>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((batch_rows_kernel<P, T, MODE, REF, A>), dim3((unsigned)nitems), dim3(256), lds, st, descs,
                     items, nitems);
  return hipGetLastError();
}

template <int KIND, int P, typename T, bool REF, typename A>
hipError_t launch_stage_of(int stage, const A &a, size_t lds, hipStream_t st) {
  switch (stage) {
    case 0: return launch_one<KIND, P, T, 0, REF>(a, lds, st);
    case 1: return launch_one<KIND, P, T, 1, REF>(a, lds, st);
    case 2:
    case 3: return launch_one<KIND, P, T, 2, REF>(a, lds, st);
    case 4: return launch_one<KIND, P, T, 4, REF>(a, lds, st);
    case kRateSums: return launch_one<KIND, P, T, kRateSums, REF>(a, lds, st);
    case kJacobian:
      if constexpr (sizeof(T) == 8) return launch_one<KIND, P, T, kJacobian, REF>(a, lds, st);
    default: return hipErrorInvalidValue;
  }
}
template <int P, typename T, bool REF, typename A>
hipError_t launch_kind(int kind, const A &a, size_t lds, hipStream_t st) {
  if (kind == kKindElement) return launch_stage_of<kKindElement, P, T, REF>(a.stage, a, lds, st);
  if (kind == kKindWave) return launch_stage_of<kKindWave, P, T, REF>(a.stage, a, lds, st);
  return hipErrorInvalidValue;
}
template <int P, typename T, bool REF, typename A>
hipError_t launch_batch_p(int stage, const A *descs, const int2 *items, int nitems, size_t lds, hipStream_t st) {
  switch (stage) {
    case kRateSums: return launch_batch_one<P, T, kRateSums, REF>(descs, items, nitems, lds, st);
    case 1: return launch_batch_one<P, T, 1, REF>(descs, items, nitems, lds, st);
    case 2:
    case 3: return launch_batch_one<P, T, 2, REF>(descs, items, nitems, lds, st);
    case 4: return launch_batch_one<P, T, 4, REF>(descs, items, nitems, lds, st);
    default: return hipErrorInvalidValue;
  }
}
template <typename T, bool REF, typename A>
hipError_t launch_batch_any(int p, int stage, const A *descs, const int2 *items, int nitems, size_t lds,
                            hipStream_t st) {
  switch (p) {
    case 1: return launch_batch_p<1, T, REF>(stage, descs, items, nitems, lds, st);
    case 2: return launch_batch_p<2, T, REF>(stage, descs, items, nitems, lds, st);
    case 3: return launch_batch_p<3, T, REF>(stage, descs, items, nitems, lds, st);
    case 4: return launch_batch_p<4, T, REF>(stage, descs, items, nitems, lds, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rows
}  // namespace dgbgk
