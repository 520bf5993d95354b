// qedx_subset.h -- building blocks of the kernels that take one current per
// photon subset, beside those of qedx_device.h.
#pragma once

namespace qx {

// acc += eps-slash J, 8 x 3 FMAs
template <class T> QEDX_HD void vL_add(sp4<T>& o, const sp4<T>& J, const pol3<T>& e) {
  const cx<T>&L0 = J.c[0], &L1 = J.c[1], &R0 = J.c[2], &R1 = J.c[3];
  o.c[0].r = o.c[0].r - e.e3 * R0.r - e.e1 * R1.r - e.e2 * R1.i;
  o.c[0].i = o.c[0].i - e.e3 * R0.i - e.e1 * R1.i + e.e2 * R1.r;
  o.c[1].r = o.c[1].r - e.e1 * R0.r + e.e2 * R0.i + e.e3 * R1.r;
  o.c[1].i = o.c[1].i - e.e1 * R0.i - e.e2 * R0.r + e.e3 * R1.i;
  o.c[2].r = o.c[2].r + e.e3 * L0.r + e.e1 * L1.r + e.e2 * L1.i;
  o.c[2].i = o.c[2].i + e.e3 * L0.i + e.e1 * L1.i - e.e2 * L1.r;
  o.c[3].r = o.c[3].r + e.e1 * L0.r - e.e2 * L0.i - e.e3 * L1.r;
  o.c[3].i = o.c[3].i + e.e1 * L0.i + e.e2 * L0.r - e.e3 * L1.i;
}
// The same for the polarisation across the z axis, e3 = 0: 8 x 2 FMAs
template <class T> QEDX_HD void vL_add_flat(sp4<T>& o, const sp4<T>& J, T e1, T e2) {
  const cx<T>&L0 = J.c[0], &L1 = J.c[1], &R0 = J.c[2], &R1 = J.c[3];
  o.c[0].r = o.c[0].r - e1 * R1.r - e2 * R1.i;
  o.c[0].i = o.c[0].i - e1 * R1.i + e2 * R1.r;
  o.c[1].r = o.c[1].r - e1 * R0.r + e2 * R0.i;
  o.c[1].i = o.c[1].i - e1 * R0.i - e2 * R0.r;
  o.c[2].r = o.c[2].r + e1 * L1.r + e2 * L1.i;
  o.c[2].i = o.c[2].i + e1 * L1.i - e2 * L1.r;
  o.c[3].r = o.c[3].r + e1 * L0.r - e2 * L0.i;
  o.c[3].i = o.c[3].i + e1 * L0.i + e2 * L0.r;
}
// The join with the row current written as the column (-B1, B0, -B3, B2):
// acc += X1 Y0 - X0 Y1 + X3 Y2 - X2 Y3 (antisymmetric in X, Y).        32 FLOPs
template <class T> QEDX_HD void pair_acc(cx<T>& acc, const sp4<T>& X, const sp4<T>& Y) {
  T r = acc.r, i = acc.i;
#pragma unroll
  for (int k = 0; k < 4; k += 2) {
    const cx<T>&x0 = X.c[k], &x1 = X.c[k + 1], &y0 = Y.c[k], &y1 = Y.c[k + 1];
    r = r + x1.r * y0.r - x0.r * y1.r - x1.i * y0.i + x0.i * y1.i;
    i = i + x1.r * y0.i - x0.r * y1.i + x1.i * y0.r - x0.i * y1.r;
  }
  acc.r = r;
  acc.i = i;
}
// Propagator of the electron p with the photons K (s = 1: Q = p + K, s = -1:
// p - K) in units of m: the column (Q-slash + 1) X, without its factor 1/D
// where one scalar can take it.  Q-slash X adds to X, so no coefficient is
// divided by D: 24 FMAs and 8 multiplications with 1/D.
template <class T> QEDX_HD sp4<T> prop_num(const sp4<T>& X, T p0, T p1, T p2, T p3, T K0, T K1, T K2, T K3, T s, T& id) {
  const T pK = p0 * K0 - p1 * K1 - p2 * K2 - p3 * K3;
  const T KK = K0 * K0 - K1 * K1 - K2 * K2 - K3 * K3;
  id = rcp(2.0 * s * pK + KK);
  const T Q0 = p0 + s * K0, Q1 = p1 + s * K1, Q2 = p2 + s * K2, Q3 = p3 + s * K3, qm = Q0 - Q3, qp = Q0 + Q3;
  const cx<T>&L0 = X.c[0], &L1 = X.c[1], &R0 = X.c[2], &R1 = X.c[3];
  sp4<T> o;
  o.c[0].r = L0.r + qm * R0.r - Q1 * R1.r - Q2 * R1.i;
  o.c[0].i = L0.i + qm * R0.i - Q1 * R1.i + Q2 * R1.r;
  o.c[1].r = L1.r - Q1 * R0.r + Q2 * R0.i + qp * R1.r;
  o.c[1].i = L1.i - Q1 * R0.i - Q2 * R0.r + qp * R1.i;
  o.c[2].r = R0.r + qp * L0.r + Q1 * L1.r + Q2 * L1.i;
  o.c[2].i = R0.i + qp * L0.i + Q1 * L1.i - Q2 * L1.r;
  o.c[3].r = R1.r + Q1 * L0.r - Q2 * L0.i + qm * L1.r;
  o.c[3].i = R1.i + Q1 * L0.i + Q2 * L0.r + qm * L1.i;
  return o;
}
template <class T> QEDX_HD sp4<T> scaled(const sp4<T>& X, T f) {
  sp4<T> o;
#pragma unroll
  for (int k = 0; k < 4; ++k) o.c[k] = {X.c[k].r * f, X.c[k].i * f};
  return o;
}
// A row adjoint in the column form of its electron line: (-w1, w0, -w3, w2).
template <class T> QEDX_HD sp4<T> as_column(const sp4<T>& w) {
  sp4<T> o;
  o.c[0] = {-w.c[1].r, -w.c[1].i};
  o.c[1] = w.c[0];
  o.c[2] = {-w.c[3].r, -w.c[3].i};
  o.c[3] = w.c[2];
  return o;
}
// Re(w Q-slash C) = Q0 bil0(w, C) + Q . bil3(w, C), w a row in column form.
// 8 and 24 FMAs.
template <class T> QEDX_HD pol3<T> bil3(const sp4<T>& w, const sp4<T>& J) {
  const cx<T>&a = w.c[0], &b = w.c[1], &c = w.c[2], &d = w.c[3];
  const cx<T>&L0 = J.c[0], &L1 = J.c[1], &R0 = J.c[2], &R1 = J.c[3];
  pol3<T> g;
  g.e1 = a.r * R0.r - a.i * R0.i - b.r * R1.r + b.i * R1.i + d.r * L1.r - d.i * L1.i - c.r * L0.r + c.i * L0.i;
  g.e2 = d.r * L1.i + d.i * L1.r + c.r * L0.i + c.i * L0.r - b.r * R1.i - b.i * R1.r - a.r * R0.i - a.i * R0.r;
  g.e3 = d.r * L0.r - d.i * L0.i + c.r * L1.r - c.i * L1.i - b.r * R0.r + b.i * R0.i - a.r * R1.r + a.i * R1.i;
  return g;
}
template <class T> QEDX_HD T bil0(const sp4<T>& w, const sp4<T>& J) {
  const cx<T>&a = w.c[0], &b = w.c[1], &c = w.c[2], &d = w.c[3];
  return b.r * J.c[2].r - b.i * J.c[2].i - a.r * J.c[3].r + a.i * J.c[3].i + d.r * J.c[0].r - d.i * J.c[0].i -
         c.r * J.c[1].r + c.i * J.c[1].i;
}

#if defined(__HIP_DEVICE_COMPILE__)
// A current in a wave's LDS region: component k of every lane at p[64 k]
// (p already offset by the lane), 16 bytes per lane and access.
__device__ inline void cur_put(double2* p, const sp4<double>& x) {
#pragma unroll
  for (int k = 0; k < 4; ++k) p[64 * k] = make_double2(x.c[k].r, x.c[k].i);
}
__device__ inline sp4<double> cur_get(const double2* p) {
  sp4<double> x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double2 t = p[64 * k];
    x.c[k] = {t.x, t.y};
  }
  return x;
}

// Shared-current kernels: component k of a current at p[NC k]; polarisation
// vector i of NP in NP pairs (e1, e2) and the NP e3 after them; propagator
// coefficients at p[0], p[D], p[2 D].
template <int NC> __device__ inline sp4<double> cur_at(const double2* p) {
  sp4<double> x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double2 t = p[NC * k];
    x.c[k] = {t.x, t.y};
  }
  return x;
}
template <int NC> __device__ inline void cur_to(double2* p, const sp4<double>& x) {
#pragma unroll
  for (int k = 0; k < 4; ++k) p[NC * k] = make_double2(x.c[k].r, x.c[k].i);
}
template <int NP> __device__ inline pol3<double> pol_at(const double2* p, unsigned i) {
  const double2 a = p[i];
  return {a.x, a.y, ((const double*)(p + NP))[i]};
}
template <int D> __device__ inline propq<double> prop_at(const double2* p) {
  const double2 a = p[0], b = p[D];
  return {a.x, a.y, b.x, b.y, p[2 * D].x};
}
// The value of the even (0) or odd (1) lane of a pair, on both.
template <int I> __device__ inline double lane_of_pair(double x) {
  const long long v = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, I ? 0xF5 : 0xA0, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), I ? 0xF5 : 0xA0, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (long long)(unsigned)lo | (long long)hi << 32);
}
// Copies a dword per lane, at offset `at` from a uniform address, to 256 bytes
// of LDS without a register.  The wave
// waits for the copies with lds_arrived() and, before the next ones, for its
// own reads with lds_taken().
__device__ inline void to_lds(const char* src, unsigned at, double* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned*)(src + at),
                                   (__attribute__((address_space(3))) unsigned*)dst, 4, 0, 0);
}
__device__ inline void lds_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ inline void lds_taken() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// Orders the wave's LDS accesses (the hardware keeps them in program order).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Workgroups go round the 8 XCDs in turn; neighbouring tiles, which share
// cache lines of the momenta, are kept on one XCD and its L2.
__device__ inline long long xcd_tile() {
  const unsigned n = gridDim.x, per = (n + 7u) >> 3, full = n & 7u;
  const unsigned x = blockIdx.x & 7u, i = blockIdx.x >> 3;
  // XCDs below `full` (all of them if it is 0) hold per tiles, the others per - 1
  const unsigned lo = full == 0u || x <= full ? x * per : full * per + (x - full) * (per - 1u);
  return (long long)lo + i;
}
#endif

}  // namespace qx
