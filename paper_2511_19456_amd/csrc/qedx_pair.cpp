// qedx_pair.cpp -- see qedx_pair.hpp.
#include "qedx_pair.hpp"

#include <map>
#include <sstream>
#include <vector>

namespace qedx {
namespace {

int popc(uint32_t x) { return __builtin_popcount(x); }

// Subsets of size k of P photons in increasing order.
std::vector<uint32_t> subsets(int P, int k) {
  std::vector<uint32_t> s;
  for (uint32_t m = 0; m < (1u << P); ++m)
    if (popc(m) == k) s.push_back(m);
  return s;
}

// 7 photons: slots of the wave's LDS region for three-photon currents (16
// bytes x 4 per lane each), before the photon momenta of its 32 points
constexpr int kSlots = 8;

struct Body {
  const Process& pr;
  std::ostringstream os;
  EmitStats st;
  std::map<uint32_t, int> slot;  // subset -> LDS slot of its current
  int h;                         // photons per side of the join (odd P: the middle photon apart)
  bool lds;                      // photon momenta and some currents in LDS

  explicit Body(const Process& p) : pr(p), h(p.P / 2), lds(pair_lds_doubles(p) > 0) {}

  std::string J(uint32_t m) const { return "J" + std::to_string(m); }

  void K(uint32_t m, const std::string& nm) {
    for (int mu = 0; mu < 4; ++mu) {
      os << "  const double " << nm << mu << " = ";
      bool first = true;
      for (int a = 0; a < pr.P; ++a)
        if ((m >> a) & 1) {
          const bool neg = pr.photon_sign[a] < 0;
          os << (first ? (neg ? "-" : "") : (neg ? " - " : " + "));
          if (lds)
            os << "lds[ko + " << 512 * kSlots + (4 * a + mu) * 32 << "]";
          else
            os << "k" << a << "_" << mu;
          first = false;
        }
      os << ";\n";
    }
    st.flops_per_point += 4.0 * (popc(m) - 1);
  }
  // The lane's offsets into the LDS region, opaque: what is kept there is read
  // back in each block of the join instead of being forwarded in registers.
  void open() {
    os << "  {\n";
    if (lds)
      os << "  unsigned go = __lane_id(), ko = __lane_id() >> 1;\n  asm volatile(\"\" : \"+v\"(go), \"+v\"(ko));\n";
  }
  std::string get(uint32_t m) const {
    auto it = slot.find(m);
    return it == slot.end() ? J(m) : "qx::cur_get((const double2*)lds + (go + " + std::to_string(256 * it->second) + "))";
  }
  // J = S(Q) X.  One current after the other where they fill the registers:
  // the scheduler, waiting for 1/D, keeps several under way and spills (6
  // photons 478 us without the barriers, 350 with them).  With 7 photons the
  // coefficients are divided by D instead, which keeps less under way than the
  // undivided current (62 instead of 87 registers spilled in the batch kernel,
  // the n = 1..6 batch 788 instead of 828 us).
  void current(uint32_t m) {
    vertices(m, "X" + std::to_string(m));
    const std::string n = std::to_string(m);
    if (pr.P >= 7) {
      os << "  qx::sp4<double> " << J(m) << ";\n  {\n";
      K(m, "K");
      os << "  " << J(m) << " = qx::sL<double>(X" << n << ", qx::prop_from<double>(pe0, pe1, pe2, pe3, K0, K1, K2, K3, sd, 1.0));\n  }\n";
      st.flops_per_point += 28 + 56;
      ++st.n_prop;
      ++st.n_S1;
    } else {
      prop(m, "Y" + n, "X" + n, "i" + n);
      os << "  const qx::sp4<double> " << J(m) << " = qx::scaled<double>(Y" << n << ", i" << n << ");\n";
      st.flops_per_point += 8;
    }
    if (pr.P >= 6) os << "  __builtin_amdgcn_sched_barrier(0);\n";
  }
  // Y = D S(Q) X, i = 1/D
  void prop(uint32_t m, const std::string& Y, const std::string& X, const std::string& i) {
    os << "  qx::sp4<double> " << Y << ";\n  double " << i << ";\n  {\n";
    K(m, "K");
    os << "  " << Y << " = qx::prop_num<double>(" << X << ", pe0, pe1, pe2, pe3, K0, K1, K2, K3, sd, " << i << ");\n  }\n";
    st.flops_per_point += 28 + 48;
    ++st.n_prop;
    ++st.n_S1;
  }
  // X = sum over a in m of eps_a-slash J(m \ a)
  void vertices(uint32_t m, const std::string& X) {
    bool first = true;
    for (int a = 0; a < pr.P; ++a) {
      if (!((m >> a) & 1)) continue;
      const uint32_t r = m & ~(1u << a);
      if (first)
        os << "  qx::sp4<double> " << X << " = qx::vL<double>(" << J(r) << ", e" << a << ");\n";
      else
        os << "  qx::vL_add<double>(" << X << ", " << J(r) << ", e" << a << ");\n";
      st.flops_per_point += first ? 40 : 48;
      ++st.n_V;
      first = false;
    }
  }

  void build() {
    const int P = pr.P;
    os << "  const unsigned q = __lane_id() & 1u;\n";
    os << "  const double sd = q ? -1.0 : 1.0;\n";
    os << "  const unsigned hc = in.hel;\n";
    os << "  const double pe0 = in.pe[0], pe1 = in.pe[1], pe2 = in.pe[2], pe3 = in.pe[3];\n";
    for (int a = 0; a < P; ++a)
      for (int mu = 0; mu < 4; ++mu)
        os << "  const double k" << a << "_" << mu << " = in.k[" << a << "][" << mu << "];\n";
    if (lds) {
      os << "  const unsigned go = __lane_id(), ko = __lane_id() >> 1;\n";
      for (int a = 0; a < P; ++a)
        for (int mu = 0; mu < 4; ++mu)
          os << "  lds[ko + " << 512 * kSlots + (4 * a + mu) * 32 << "] = k" << a << "_" << mu << ";\n";
    }
    // the lanes' polarisation vectors are the same: each computes half and takes the rest from its partner
    for (int a = 0; a + 1 < P; a += 2) {
      os << "  qx::pol3<double> e" << a << ", e" << a + 1 << ";\n  {\n";
      os << "    const qx::pol3<double> o = qx::pol<double>(q ? k" << a + 1 << "_1 : k" << a << "_1, q ? k" << a + 1
         << "_2 : k" << a << "_2, q ? k" << a + 1 << "_3 : k" << a << "_3, (int)((hc >> (q ? "
         << pr.photon_particle[a + 1] << "u : " << pr.photon_particle[a] << "u)) & 1u));\n";
      for (int i = 0; i < 2; ++i)
        for (int c = 1; c < 4; ++c)
          os << "    e" << a + i << ".e" << c << " = qx::lane_of_pair<" << i << ">(o.e" << c << ");\n";
      os << "  }\n";
      st.flops_per_point += 16;
    }
    if (P % 2) {
      const int a = P - 1;
      os << "  const qx::pol3<double> e" << a << " = qx::pol<double>(k" << a << "_1, k" << a << "_2, k" << a
         << "_3, (int)((hc >> " << pr.photon_particle[a] << ") & 1u));\n";
      st.flops_per_point += 16;
    }
    st.n_U = 2 + P;
    os << "  const qx::sp4<double> J0 = qx::u_in<double>(pe0, pe1, pe2, pe3, (int)(((hc >> (q ? " << pr.i_eout << "u : "
       << pr.i_ein << "u)) & 1u) ^ q), 1.0);\n";
    st.flops_per_point += 16;
    // propagated currents of every subset below the join; with 7 photons the
    // three-photon ones without the last photon wait for the join
    const int top_k = P % 2 ? h : h - 1;
    const uint32_t last = 1u << (P - 1);
    for (int k = 1; k <= top_k; ++k)
      for (uint32_t m : subsets(P, k)) {
        if (lds && k == 3 && !(m & last)) continue;
        current(m);
        if (lds && k == 3 && (int)slot.size() < kSlots) {
          const int n = (int)slot.size();
          slot[m] = n;
          os << "  qx::cur_put((double2*)lds + (go + " << 256 * n << "), " << J(m) << ");\n";
        }
      }
    os << "  qx::cx<double> A = {0.0, 0.0};\n";
    const uint32_t full = (1u << P) - 1;
    if (P % 2 == 0) {
      // each unordered pair of complementary subsets is two partitions: a
      // lane propagates its current of one subset and joins it to the partner's of the other
      for (uint32_t m : subsets(P, h)) {
        if (!(m & 1)) continue;
        open();
        vertices(full & ~m, "C");
        os << "  const qx::sp4<double> R = qx::lane_xor1(C);\n";
        vertices(m, "X");
        prop(m, "Y", "X", "i");
        os << "  qx::cx<double> B = {0.0, 0.0};\n  qx::pair_acc<double>(B, R, Y);\n  A.r += i * B.r;\n  A.i += i * B.i;\n  }\n";
        st.flops_per_point += 36;
        ++st.n_dot;
      }
    } else {
      // two disjoint subsets of h photons and the photon a between them: the
      // lane applies eps_a to its current of one and joins it to the
      // partner's of the other.  Every unordered pair is taken once, grouped
      // by the received subset r (those without the last photon meet every pair).
      auto join = [&](uint32_t r, bool with_complement) {
        os << "  {\n";
        bool first = true;
        for (uint32_t s : subsets(P, h)) {
          if ((s & r) || (!(s & last) && !with_complement)) continue;
          const int a = __builtin_ctz(full & ~(s | r));
          if (first)
            os << "  qx::sp4<double> Y = qx::vL<double>(" << get(s) << ", e" << a << ");\n";
          else
            os << "  qx::vL_add<double>(Y, " << get(s) << ", e" << a << ");\n";
          st.flops_per_point += first ? 40 : 48;
          ++st.n_V;
          first = false;
        }
        os << "  qx::pair_acc<double>(A, qx::lane_xor1(" << J(r) << "), Y);\n  }\n";
        st.flops_per_point += 32;
        ++st.n_dot;
      };
      // among the subsets without the last photon only r and full \ r \ last are disjoint
      for (uint32_t r : subsets(P, h)) {
        if (r & last) continue;
        const uint32_t rc = full & ~last & ~r;
        if (h > 1 && !(r & 1)) continue;
        open();
        if (lds) {
          current(r);
          current(rc);
        }
        join(r, h > 1 || r == 1);
        if (h > 1) join(rc, false);
        os << "  }\n";
      }
    }
    // the join's form is antisymmetric: the e-_out lane's share carries a minus sign
    os << "  A.r *= sd;\n  A.i *= sd;\n";
    os << "  A.r += qx::lane_xor1(A.r);\n  A.i += qx::lane_xor1(A.i);\n";
    os << "  return A.r * A.r + A.i * A.i;\n";
    st.flops_per_point = 2 * (st.flops_per_point + 7);  // both lanes
  }
};

}  // namespace

int pair_lds_doubles(const Process& pr) { return pr.P >= 7 ? 512 * kSlots + 32 * 4 * pr.P : 0; }

int pair_in_doubles(const Process& pr) { return pair_persistent(pr) ? 32 * (4 * pr.npart + 1) : 0; }

int pair_waves(const Process& pr) { return pr.P >= 5 ? 1 : 2; }

// 7 photons: a workgroup of four waves would hold the whole LDS until its last
// wave ends; single waves make way as they end (64 points 30.1 -> 28.0 us, 10^6
// points 968 -> 914 us).
int pair_block(const Process& pr) { return pair_lds_doubles(pr) > 0 ? 64 : 256; }

bool pair_persistent(const Process& pr) { return pr.P == 5 || pr.P == 6; }

std::string emit_pair_body(const Process& pr, const std::string& fname, EmitStats* st) {
  Body b(pr);
  b.build();
  if (st) *st = b.st;
  std::ostringstream os;
  // a lane's inputs: its electron's momentum, the photons', the helicity code
  os << "struct " << fname << "_in { double pe[4], k[" << pr.P << "][4]; unsigned hel; };\n";
  os << "static __device__ __forceinline__ void " << fname
     << "_load(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, long long pt, " << fname
     << "_in& in)\n{\n";
  os << "  const double* const pm = mom + ((__lane_id() & 1u) ? " << 4 * pr.i_eout << "LL : " << 4 * pr.i_ein
     << "LL) * N + pt;\n  const double* const pk = mom + pt;\n  in.hel = hel[pt];\n";
  os << "#pragma unroll\n  for (int mu = 0; mu < 4; ++mu) {\n    in.pe[mu] = pm[mu * N];\n";
  for (int a = 0; a < pr.P; ++a)
    os << "    in.k[" << a << "][mu] = pk[(" << 4 * pr.photon_particle[a] << " + mu) * N];\n";
  os << "  }\n}\n";
  if (pair_persistent(pr)) {
    const int R = 4 * pr.npart;
    os << "static __device__ __forceinline__ void " << fname
       << "_fetch(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, long long p0, double* buf)\n{\n"
       << "  const long long first = p0 < N ? p0 : N - 1;\n  const unsigned left = N - 1 - first < 31 ? (unsigned)(N - 1 - first) : 31u;\n"
       << "  const unsigned i = __lane_id() >> 1, j = __lane_id() & 31u;\n"
       << "  const unsigned at = 8u * (i < left ? i : left) + 4u * (__lane_id() & 1u);\n  const char* row = (const char*)(mom + first);\n"
       << "#pragma unroll 4\n  for (int r = 0; r < " << R << "; ++r, row += 8 * N) qx::to_lds(row, at, buf + 32 * r);\n"
       << "  qx::to_lds((const char*)(hel + first), 4u * (j < left ? j : left), buf + " << 32 * R << ");\n}\n";
    os << "static __device__ __forceinline__ void " << fname << "_take(const double* buf, " << fname << "_in& in)\n{\n"
       << "  const unsigned g = __lane_id() >> 1, e = (__lane_id() & 1u) ? " << 128 * pr.i_eout << "u + g : " << 128 * pr.i_ein
       << "u + g;\n  in.hel = ((const unsigned*)(buf + " << 32 * R << "))[g];\n"
       << "#pragma unroll\n  for (int mu = 0; mu < 4; ++mu) {\n    in.pe[mu] = buf[e + 32 * mu];\n";
    for (int a = 0; a < pr.P; ++a)
      os << "    in.k[" << a << "][mu] = buf[g + " << 128 * pr.photon_particle[a] << " + 32 * mu];\n";
    os << "  }\n}\n";
  }
  os << "static __device__ __forceinline__ double " << fname << "_run(const " << fname
     << "_in& in, double* __restrict__ lds)\n{\n" << b.os.str() << "}\n";
  os << "static __device__ __forceinline__ double " << fname
     << "(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, long long pt, double* "
        "__restrict__ lds)\n{\n  " << fname << "_in in;\n  " << fname << "_load(mom, hel, N, pt, in);\n  return " << fname
     << "_run(in, lds);\n}\n";
  if (!pair_persistent(pr)) return os.str();
  os << "static __device__ __forceinline__ void " << fname
     << "_tiles(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, double* __restrict__ out, long long p0, "
        "long long step, long long end, double* __restrict__ buf)\n{\n";
  os << "  if (p0 >= end) return;\n  qx::lds_taken();\n  " << fname << "_fetch(mom, hel, N, p0, buf);\n";
  os << "  long long last = -1;\n  double r = 0.0;\n  while (true) {\n    " << fname << "_in in;\n    qx::lds_arrived();\n    " << fname
     << "_take(buf, in);\n    qx::lds_taken();\n";
  os << "    const long long nx = p0 + step;\n    if (nx < end) " << fname << "_fetch(mom, hel, N, nx, buf);\n";
  os << "    if (last >= 0 && last < N && (__lane_id() & 1u) == 0u) out[last] = r;\n    __builtin_amdgcn_sched_barrier(0);\n";
  os << "    r = " << fname << "_run(in, nullptr);\n    last = p0 + (__lane_id() >> 1);\n    if (nx >= end) break;\n    p0 = nx;\n  }\n";
  os << "  if (last < N && (__lane_id() & 1u) == 0u) out[last] = r;\n}\n";
  return os.str();
}

std::string emit_pair_kernel(const Process& pr, const Variant& v, const std::string& kname, EmitStats* st) {
  std::ostringstream os;
  os << "// generated by qedx: " << variant_tag(v, pr.n_out, pr.n_in) << "\n";
  os << kContractOn << "// subset currents, lane 0 of a point from e-_in, lane 1 from e-_out\n";
  os << "#include <hip/hip_runtime.h>\n" << device_header_text() << "\n" << subset_header_text() << "\n";
  const std::string body = kname + "_body";
  os << emit_pair_body(pr, body, st);
  const int W = pair_lds_doubles(pr), B = pair_block(pr);
  os << "extern \"C\" __global__ void __launch_bounds__(" << B << ", " << pair_waves(pr) << ")\n" << kname
     << "(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, double* __restrict__ out)\n{\n";
  if (W) os << "  __shared__ double2 qx_lds[" << B / 64 * W / 2 << "];\n";
  const std::string lds = W ? "(double*)qx_lds + (threadIdx.x >> 6) * " + std::to_string(W) : std::string("nullptr");
  if (pair_persistent(pr)) {
    os << "  __shared__ double qx_in[4][" << pair_in_doubles(pr) << "];\n";
    os << "  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));\n";
    os << "  " << body << "_tiles(mom, hel, N, out, (long long)blockIdx.x * 128 + 32 * wave, 128LL * gridDim.x, N, qx_in[wave]);\n}\n";
  } else {
    os << "  const long long pt = ((long long)blockIdx.x * " << B << " + threadIdx.x) >> 1;\n";
    os << "  const double r = " << body << "(mom, hel, N, pt < N ? pt : N - 1, " << lds << ");\n";
    os << "  if (pt < N && (threadIdx.x & 1u) == 0u) out[pt] = r;\n}\n";
  }
  return os.str();
}

}  // namespace qedx
