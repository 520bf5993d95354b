// qedx_kernels.hpp -- auxiliary generated module: RAMBO and gradient kernels.
#pragma once

#include <string>

#include "qedx_dag.hpp"
#include "qedx_emit.hpp"

namespace qedx {

// Launch shapes of the auxiliary module's gradient kernels.
struct AuxInfo {
  int grad_points = 0;  // points of one wave of the gradient kernel (0: no gradient)
  int split = 0;        // 1: split gradient kernels
};

// HIP source with
//   qedx_rambo_n<n>(const double* u, double sqrt_s, long long N, double* mom)
// and, for SUM-mode FP64 processes of n <= 4, the gradient of log |M|^2 with
// respect to the RAMBO uniforms:
//  - n <= 3, fused: qedx_grad_n<n>(const double* u, double sqrt_s, long long N,
//      double* logm2, double* grad, int tiles);
//  - n = 4, split over a caller workspace (two points per wave leave no LDS for
//      the phase space of a whole wave's points):
//      qedx_grambo_n<n>(u, ldu, sqrt_s, N, mom)      RAMBO into the workspace,
//      qedx_gmom_n<n>(mom, N, gm, logm2)             momentum gradient of log |M|^2,
//      qedx_grvjp_n<n>(u, ldu, sqrt_s, N, gm, grad, ldg)  RAMBO adjoint.
// qedx_grad_low_n<n>, qedx_gmom_low_n<n>: the same for sqrt(s) below kWardFrom.
// n >= 5 has RAMBO only.
std::string emit_aux_module(const Process& proc, const Variant& v, int n, AuxInfo* info);

}  // namespace qedx
