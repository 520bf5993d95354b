// qedx_pair.hpp -- FP64 kernels for one configuration per point, two lanes
// per point.
//
// Lane 0 of a point builds the currents of the photon subsets from e-_in,
// lane 1 those from e-_out, one current per subset (the sum over the photon
// orderings is taken before the next vertex).  Written as a column through
// the antiunitary map that turns the row ubar(p', s) into the column u(p', 1 - s),
// the e-_out side obeys the same vertex and propagator with Q = p' - K in
// place of Q = p + K, so both lanes run one instruction stream on their own
// electron momentum, spin and sign of K.  The join takes half of the photon
// partitions on each lane, which hands its partner one current per pair of
// partitions (DPP lane swap).
//
// Bound by FP64 vector instructions: 1.1 (4 photons) to 12.1 (7 photons)
// thousand per lane, 0.75-0.85 of them FP64 arithmetic, against 3626 to 283306
// FLOPs of the graph that keeps the orderings apart.  Two lanes, because one
// lane's registers hold one side's currents (P = 6: 15 of 8 doubles) and not
// both.  They stay in registers up to 6 photons (vector and accumulation
// registers, one wave per SIMD): kept in LDS instead, 8 of the 15 took 408 us
// where the registers take 361 (2^20 points, P = 6).  One wave per SIMD hides
// no load, so P = 5, 6 loop over the points and copy the next ones' momenta
// into LDS while they work, which takes no register (P = 6: 445 us without
// loading ahead, 375 us into registers, 349 us into LDS; P = 5: 181, 169 and
// 162 us); P <= 4 fits 2 to 8 waves per SIMD and is faster in one pass (P = 4:
// 75 against 88 us).  P = 7 has no LDS left for that: its three-photon
// currents with the last photon go there, the others are built where the join
// needs them.
// Against one product per ordering (2^20 points): P = 5 418 -> 162 us, P = 6
// 1421 -> 349 us; P = 7, 100003 points with their phase space, 874 -> 144 us;
// the mixed n = 1..6 batch of 2.77 M points 4.62 -> 0.79 ms.  VALU busy: P = 5
// 88 %, P = 6 93 %, P = 7 67 %.
#pragma once

#include <string>

#include "qedx_dag.hpp"
#include "qedx_emit.hpp"

namespace qedx {

// Second line of the sources compiled with FMAs formed within an expression
// only: a process's eval kernel and the batch kernels of processes without a
// given shape give the same bits.  (The pair bodies of the other modules, beside
// graph bodies and in the FP64 pass of FP32C, are compiled with those and may
// differ from them in the last bits.)
constexpr const char* kContractOn = "// fp-contract: on\n";

// Whether (process, variant) takes the pair body in FP64: its eval kernel if
// it is an FP64 process, else the FP64 pass after its FP32C kernel.
inline bool pair_kernel(const Process& pr, const Variant& v) { return v.subset && v.mode == HEL_PER_POINT; }
// Whether its eval kernel does.
inline bool pair_eval(const Process& pr, const Variant& v) { return v.prec == PREC_F64 && pair_kernel(pr, v); }

// Device function text
//   static __device__ double <fname>(const double* mom, const unsigned* hel, long long N, long long pt, double* lds)
// for lanes 2i, 2i + 1 of a wave working on the same point; both return the
// point's |A|^2.  lds: the wave's region of pair_lds_doubles() doubles, 16-byte aligned.
std::string emit_pair_body(const Process& pr, const std::string& fname, EmitStats* st);
int pair_lds_doubles(const Process& pr);
// Whether the eval kernel is launched with one workgroup per compute unit and
// its waves loop over the points, by the function
//   void <fname>_tiles(mom, hel, N, out, long long p0, long long step, long long end, double* buf):
// the wave's points are the 32 from p0 on, p0 + step, ... below end; buf: the
// wave's LDS for the inputs under way, pair_in_doubles() doubles.
bool pair_persistent(const Process& pr);
int pair_in_doubles(const Process& pr);
// Threads per workgroup of the eval kernel.
int pair_block(const Process& pr);
// Waves per SIMD the body's registers and LDS are laid out for.
int pair_waves(const Process& pr);

// The eval kernel around it: extern "C" __global__ void <kname>(mom, hel, N, out).
std::string emit_pair_kernel(const Process& pr, const Variant& v, const std::string& kname, EmitStats* st);

}  // namespace qedx
