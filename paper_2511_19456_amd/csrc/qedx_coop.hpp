// qedx_coop.hpp -- FP64 helicity sums, the lanes of a point sharing its
// currents through LDS.
//
// The currents of the photon subsets are built level by level (all subsets of
// k photons, each with its 2^k polarisation configurations) from e-_in only;
// the last level holds every photon and is closed with both spins of e-_out,
// so there is no join.  The lanes of a point take the items (subset,
// configuration) of a level in turn, read the level below from LDS and write
// their own over it.  Only one spin of e-_in is built: for real polarisations
// the antiunitary map (L, R) -> (i sigma2 R*, i sigma2 L*) commutes with vertices
// and propagators and exchanges the spins u(p, 0), u(p, 1), so |A(s, s')| =
// |A(1-s, 1-s')| for any momenta, and the sum is twice the half.
//
// Two resources share the bound: FP64 vector instructions (1.35 thousand per
// lane at 4 photons, 1.55 at 5) and LDS reads (a vertex reads 88 bytes per lane
// for 24 instructions, 0.9 of the time its instructions take).  Measured
// against the kernels with one product per ordering, both spins and the joins
// (2^20 points): 4 photons 1.61 -> 0.435 ms (VALU busy 0.67, LDS 0.48), 3
// photons 407 -> 149 us, 2 photons 98 -> 50 us; 5 photons, 99991 points, 2.52 ->
// 0.170 ms (0.74, 0.53).
#pragma once

#include <string>

#include "qedx_dag.hpp"
#include "qedx_emit.hpp"

namespace qedx {

// Whether (process, variant) is evaluated by the shared-current kernels.
inline bool coop_kernel(const Process& pr, const Variant& v) {
  return v.subset && v.mode == HEL_SUM && v.prec == PREC_F64 && pr.P <= 5;
}
int coop_lanes(const Process& pr);  // lanes per point
constexpr int kCoopBlock = 64;      // one wave per workgroup

// extern "C" __global__ void <kname>(const double* mom, const unsigned* hel, long long N, double* out)
std::string emit_coop_kernel(const Process& pr, const Variant& v, const std::string& kname, EmitStats* st);

// Gradient of log sum |A|^2 for one incoming photon.  The forward levels, then
// the same levels downwards with the adjoints in the currents' LDS slots; each
// lane keeps the currents of its own items in registers (14 of them at 5
// photons), so nothing is recomputed and LDS stays what the forward needs.  The
// sums over items (28 polarisation and momentum gradients at 5 photons) are per
// lane in registers and meet in LDS once, at the end.  At 5 photons 468
// registers leave one wave per SIMD: VALU busy 0.56 of the time, LDS 0.40 (a
// fifth of that bank conflicts), 0.20 waits.  Measured against one walk over
// the orderings per partition and electron: 5 photons, 2^18 points, 14.2 -> 1.32
// ms (16 lanes per point; with 32 2.29 when 16 took 1.56); 4 photons, 2^19
// points, 48.6 -> 0.79 ms (one wave per SIMD instead of two 1.26 when two took
// 0.98); 3 photons 7.25 -> 0.28 ms, 2 photons 1.15 -> 0.16 ms.  With rambo: through the
// phase-space map,
//   <kname>(const double* u, double sqrt_s, long long N, double* logm2, double* grad, int tiles),
// one wave per `tiles` (1 .. 64 / points of a wave) groups of points; without:
//   <kname>(const double* mom, long long N, double* gm, double* logm2),
// gm the final-state rows of the momentum gradient, one group per wave.
// ward: the polarisation vectors' share through the Ward identity, for sqrt(s)
// from kWardFrom on; below it the share itself, because the identity's terms
// cancel as sqrt(s) - 1 goes to zero.  Median error of the gradient at sqrt(s)
// = 1.0001, with and without the identity, against extended precision: 2
// photons out 1.0e-8 and 4.4e-11, 4 photons 2.6e-5 and 5.3e-8; at 1.1 they are
// equal (3.4e-14, 1.5e-13) and the identity is faster: 2^18 points of 4
// photons out 1.36 against 1.47 ms, 20011 of 3 76 against 82 us.
// No device header included: the caller prepends it.
std::string emit_coop_grad_kernel(const Process& pr, const std::string& kname, bool rambo, bool ward, EmitStats* st);
constexpr double kWardFrom = 1.1;
int coop_grad_lanes(const Process& pr);

}  // namespace qedx
