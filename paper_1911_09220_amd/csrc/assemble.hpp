// Launchers of the assembly kernels on the apply's tiles (k_assemble.hip); hexahedra.
#pragma once

#include <hip/hip_runtime_api.h>

#include "internal.hpp"

namespace pafem {

// quadrature data of any kind and any q1d with a table (1..kMaxQ1d); status[0] receives
// the smallest caller element with det J <= 0
void launch_qdata_tiles(const DevSpace& sp, int kind, int q1d, const double* coeff, double scale,
                        double* qd, hipStream_t st);
// element diagonals ye [ne][(p+1)^3] of an operator with q1d = p + 2 (every operator)
void launch_diagonal_tiles(const DevSpace& sp, int kind, const double* qd, double* ye,
                           hipStream_t st);
// element load vectors for q1d = p + 2
void launch_linear_form_tiles(const DevSpace& sp, int source, const double* fqp, double scale,
                              double* ye, hipStream_t st);

}  // namespace pafem
