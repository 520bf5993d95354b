// qedx_kernels.cpp -- auxiliary generated module (RAMBO; gradient).
#include "qedx_kernels.hpp"

#include "qedx_coop.hpp"

#include <sstream>

namespace qedx {

std::string emit_aux_module(const Process& proc, const Variant& v, int n, AuxInfo* info) {
  std::ostringstream os;
  const int NF = n + 1;
  const std::string ns = std::to_string(n);
  AuxInfo ai;
  os << "// generated by qedx: auxiliary kernels for n = " << n << "\n";
  os << "#include <hip/hip_runtime.h>\n";
  os << device_header_text() << "\n";
  os << "extern \"C\" __global__ void __launch_bounds__(256)\nqedx_rambo_n" << n << "(const double* __restrict__ u, double sqrt_s, "
        "long long N, double* __restrict__ mom)\n{\n";
  os << "  const long long pt = (long long)blockIdx.x * 256 + threadIdx.x;\n";
  os << "  if (pt >= N) return;\n";
  os << "  double uu[" << 4 * NF << "];\n";
  os << "#pragma unroll\n  for (int r = 0; r < " << 4 * NF << "; ++r) uu[r] = u[r * N + pt];\n";
  os << "  qx::RamboState<" << NF << "> S;\n";
  os << "  qx::rambo_forward<" << NF << ">(uu, sqrt_s, 1.0, S);\n";
  os << "  double pin[4], kin[4];\n  qx::incoming_cm(sqrt_s, 1.0, pin, kin);\n";
  os << "#pragma unroll\n  for (int d = 0; d < 4; ++d) { mom[d * N + pt] = pin[d]; mom[(4 + d) * N + pt] = kin[d]; }\n";
  os << "#pragma unroll\n  for (int j = 0; j < " << NF << "; ++j)\n#pragma unroll\n    for (int d = 0; d < 4; ++d) mom[(4 * (2 + j) + d) * N + pt] = S.k[j][d];\n";
  os << "}\n";
  if (v.mode != HEL_SUM || v.prec != PREC_F64 || n > 4) {
    if (info) *info = ai;
    return os.str();
  }
  os << subset_header_text() << "\n";
  EmitStats st;
  ai.grad_points = 64 / coop_grad_lanes(proc);
  if (n <= 3) {
    // fused: RAMBO, currents, reverse sweep and RAMBO adjoint in one kernel
    os << emit_coop_grad_kernel(proc, "qedx_grad_n" + ns, true, true, &st);
    os << emit_coop_grad_kernel(proc, "qedx_grad_low_n" + ns, true, false, &st);
  } else {
    // split: RAMBO into the workspace, the gradient over its momenta, RAMBO adjoint
    ai.split = 1;
    os << emit_coop_grad_kernel(proc, "qedx_gmom_n" + ns, false, true, &st);
    os << emit_coop_grad_kernel(proc, "qedx_gmom_low_n" + ns, false, false, &st);
    os << "extern \"C\" __global__ void __launch_bounds__(256)\nqedx_grambo_n" << n
       << "(const double* __restrict__ u, long long ldu, double sqrt_s, long long N, double* __restrict__ mom)\n{\n";
    os << "  const long long pt = (long long)blockIdx.x * 256 + threadIdx.x;\n";
    os << "  if (pt >= N) return;\n";
    os << "  double uu[" << 4 * NF << "];\n";
    os << "#pragma unroll\n  for (int r = 0; r < " << 4 * NF << "; ++r) uu[r] = u[r * ldu + pt];\n";
    os << "  qx::RamboState<" << NF << "> S;\n";
    os << "  qx::rambo_forward<" << NF << ">(uu, sqrt_s, 1.0, S);\n";
    os << "  double pin[4], kin[4];\n  qx::incoming_cm(sqrt_s, 1.0, pin, kin);\n";
    os << "#pragma unroll\n  for (int d = 0; d < 4; ++d) { mom[d * N + pt] = pin[d]; mom[(4 + d) * N + pt] = kin[d]; }\n";
    os << "#pragma unroll\n  for (int j = 0; j < " << NF << "; ++j)\n#pragma unroll\n    for (int d = 0; d < 4; ++d) mom[(4 * (2 + j) + d) * N + pt] = S.k[j][d];\n";
    os << "}\n";
    os << "extern \"C\" __global__ void __launch_bounds__(256)\nqedx_grvjp_n" << n
       << "(const double* __restrict__ u, long long ldu, double sqrt_s, long long N, const double* __restrict__ gm, "
          "double* __restrict__ grad, long long ldg)\n{\n";
    os << "  const long long pt = (long long)blockIdx.x * 256 + threadIdx.x;\n";
    os << "  if (pt >= N) return;\n";
    os << "  double uu[" << 4 * NF << "];\n";
    os << "#pragma unroll\n  for (int r = 0; r < " << 4 * NF << "; ++r) uu[r] = u[r * ldu + pt];\n";
    os << "  qx::RamboState<" << NF << "> S;\n";
    os << "  qx::rambo_forward<" << NF << ">(uu, sqrt_s, 1.0, S);\n";
    os << "  double gk[" << NF << "][4];\n";
    os << "#pragma unroll\n  for (int j = 0; j < " << NF << "; ++j)\n#pragma unroll\n    for (int d = 0; d < 4; ++d) gk[j][d] = gm[(4 * (2 + j) + d) * N + pt];\n";
    os << "  double gu[" << 4 * NF << "];\n#pragma unroll\n  for (int r = 0; r < " << 4 * NF << "; ++r) gu[r] = 0.0;\n";
    os << "  qx::rambo_vjp<" << NF << ">(uu, sqrt_s, 1.0, S, gk, gu);\n";
    os << "#pragma unroll\n  for (int r = 0; r < " << 4 * NF << "; ++r) grad[r * ldg + pt] = gu[r];\n";
    os << "}\n";
  }
  if (info) *info = ai;
  return os.str();
}

}  // namespace qedx
