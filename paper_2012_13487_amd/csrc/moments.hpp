// Density and velocity at every node of an element-major state f[k][q][n].
#pragma once

#include <hip/hip_runtime.h>

namespace dgbgk {

// rho, ux, uy (K Np values each) of f = fd + fs + w_q offset in FP64; fd or fs
// may be null.  Np <= 256.
hipError_t launch_node_moments(const double *fd, const float *fs, double offset, const double *vel, int K, int Np,
                               int Q, double *rho, double *ux, double *uy, hipStream_t stream);

}  // namespace dgbgk
