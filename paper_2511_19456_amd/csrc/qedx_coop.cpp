// qedx_coop.cpp -- see qedx_coop.hpp.
#include "qedx_coop.hpp"

#include <algorithm>
#include <sstream>
#include <stdexcept>
#include <vector>

namespace qedx {
namespace {

int popc(uint32_t x) { return __builtin_popcount(x); }

std::vector<uint32_t> subsets(int P, int k) {
  std::vector<uint32_t> s;
  for (uint32_t m = 0; m < (1u << P); ++m)
    if (popc(m) == k) s.push_back(m);
  return s;
}

struct Coop {
  const Process& pr;
  const int P, L, PPW;
  std::ostringstream os;
  EmitStats st;
  int NC = 0, NS, pol0, prop0, PT;  // LDS of a point, in 16-byte units
  std::vector<std::vector<uint32_t>> lv;
  std::vector<std::vector<int>> index;  // index[k][mask]: position of a subset in its level
  std::vector<uint32_t> order;          // the photon subsets below the full one, by size

  explicit Coop(const Process& p) : pr(p), P(p.P), L(coop_lanes(p)), PPW(64 / L) {
    for (int k = 0; k <= P; ++k) {
      lv.push_back(subsets(P, k));
      index.push_back(std::vector<int>(1u << P, -1));
      for (size_t i = 0; i < lv[k].size(); ++i) index[k][lv[k][i]] = (int)i;
    }
    for (int k = 1; k < P; ++k) {
      NC = std::max(NC, items(k));
      order.insert(order.end(), lv[k].begin(), lv[k].end());
    }
    NS = (int)order.size();
    pol0 = 4 * NC;
    prop0 = pol0 + 3 * P;
    PT = prop0 + (overlay() ? 0 : 3 * NS);
    // lanes of neighbouring points start in different banks (16 x 16 bytes)
    while (PPW > 1 && PT % 16 != L % 16) ++PT;
  }
  int items(int k) const { return (int)lv[k].size() << k; }
  int rounds(int k) const { return (items(k) + L - 1) / L; }

  // 4 photons on 8 lanes: the propagator coefficients lie in the currents'
  // slots that are still free when they are read (2.2 instead of 2.9 KB per
  // point: two waves per SIMD)
  bool overlay() const { return P == 4 && L == 8; }
  // position of the coefficients of order[i], and the step between their three parts
  int prop_at(int i) const {
    if (!overlay()) return prop0 + i;
    return i < 4 ? 8 + i : i < 12 ? 24 + i - 4 : 3 * NC + 24 + 3 * (i - 12);
  }
  int prop_step(int i) const { return !overlay() ? NS : i < 12 ? NC : 1; }
  int order_of(uint32_t S) const { return (int)(std::find(order.begin(), order.end(), S) - order.begin()); }

  // v[(lane in point) >> k] for the m entries of v
  std::string sel(const std::vector<int>& v, int k) const {
    bool same = true;
    for (int x : v) same = same && x == v[0];
    if (same) return std::to_string(v[0]) + "u";
    const std::string i = "(l >> " + std::to_string(k) + ")";
    if (v.size() == 2) return "(" + i + " ? " + std::to_string(v[1]) + "u : " + std::to_string(v[0]) + "u)";
    // at most 8 entries, or all the same from the 8th on
    const std::string j = v.size() > 8 ? "(" + i + " < 7u ? " + i + " : 7u)" : i;
    unsigned long long w = 0;
    for (size_t t = 0; t < v.size(); ++t) {
      if (t > 7) {
        if (v[t] != v[7]) throw std::logic_error("coop: too many subsets in a round");
        continue;
      }
      if (v[t] < 0 || v[t] > 255) throw std::logic_error("coop: table entry");
      w |= (unsigned long long)v[t] << (8 * t);
    }
    return "((unsigned)(" + std::to_string(w) + "ull >> (8u * " + j + ")) & 255u)";
  }
  void sync() { os << "  qx::wave_sync();\n"; }
  std::string get(const std::string& c) const {
    return "qx::cur_at<" + std::to_string(NC) + ">(cu + (" + c + "))";
  }

  void prologue() {
    const int ein = pr.i_ein, eout = pr.i_eout;
    os << "  const unsigned l = threadIdx.x & " << L - 1 << "u;\n";
    os << "  double2* const cu = lds + (threadIdx.x / " << L << "u) * " << PT << "u;\n";
    for (int mu = 0; mu < 4; ++mu)
      os << "  const double p" << mu << " = mom[" << 4 * ein + mu << " * N + ptc], o" << mu << " = mom[" << 4 * eout + mu
         << " * N + ptc];\n";
    for (int a = 0; a < P; ++a)
      for (int mu = 0; mu < 4; ++mu)
        os << "  const double k" << a << "_" << mu << " = " << (pr.photon_sign[a] < 0 ? "-" : "") << "mom["
           << 4 * pr.photon_particle[a] + mu << " * N + ptc];\n";
    // polarisation vectors: item 2 a + lambda
    for (int r = 0; r * L < 2 * P; ++r) {
      os << "  {\n    const unsigned i = " << r * L << "u + l < " << 2 * P << "u ? " << r * L << "u + l : " << 2 * P - 1
         << "u;\n    const unsigned a = i >> 1;\n";
      for (int mu = 1; mu < 4; ++mu) {
        os << "    const double x" << mu << " = ";
        for (int a = 0; a + 1 < P; ++a) os << "a == " << a << "u ? k" << a << "_" << mu << " : ";
        os << "k" << P - 1 << "_" << mu << ";\n";
      }
      os << "    const double s = ";
      for (int a = 0; a + 1 < P; ++a) os << "a == " << a << "u ? " << pr.photon_sign[a] << ".0 : ";
      os << pr.photon_sign[P - 1] << ".0;\n";
      os << "    const qx::pol3<double> e = qx::pol<double>(s * x1, s * x2, s * x3, (int)(i & 1u));\n";
      os << "    cu[" << pol0 << "u + i] = make_double2(e.e1, e.e2);\n    ((double*)(cu + " << pol0 + 2 * P
         << "u))[i] = e.e3;\n  }\n";
      st.flops_per_point += 16.0 * L;
    }
    // propagator coefficients of every photon subset, from the electron with
    // the fewer photons (Q = p + K, or p' - K with K of the other photons):
    // Q^2 - m^2 = +-2 p.K + K^2 cancels where the photons left to the other
    // electron are soft
    int near = 0;  // order[0 .. near): counted from e-_in
    while (near < NS && 2 * popc(order[near]) <= P) ++near;
    for (int r = 0; r * L < NS; ++r) {
      const bool part = (r + 1) * L > NS;
      os << "  {\n    const unsigned i = " << r * L << "u + l;\n";
      // the subset's bits, a nibble or a byte each
      const int w = P <= 4 ? 4 : 8, per = 64 / w;
      os << "    const unsigned S = (unsigned)(";
      for (int t = 0; t * per < L; ++t) {
        unsigned long long x = 0;
        for (int j = 0; j < per; ++j)
          {
            const int i = std::min(r * L + t * per + j, NS - 1);
            x |= (unsigned long long)(i < near ? order[i] : ((1u << P) - 1) & ~order[i]) << (w * j);
          }
        if (t) os << " : ";
        if ((t + 1) * per < L) os << "l < " << (t + 1) * per << "u ? ";
        os << "(" << x << "ull >> (" << w << "u * (l & " << per - 1 << "u)))";
      }
      os << ");\n";
      for (int a = 0; a < P; ++a) os << "    const double b" << a << " = (double)((S >> " << a << ") & 1u);\n";
      for (int mu = 0; mu < 4; ++mu) {
        os << "    const double K" << mu << " = ";
        for (int a = 0; a < P; ++a) os << (a ? " + " : "") << "b" << a << " * k" << a << "_" << mu;
        os << ";\n";
      }
      if (near >= (r + 1) * L || near <= r * L) {
        const bool in = near > r * L;
        const std::string e = in ? "p" : "o";
        os << "    const qx::propq<double> q = qx::prop_from<double>(" << e << "0, " << e << "1, " << e << "2, " << e
           << "3, K0, K1, K2, K3, " << (in ? "1.0" : "-1.0") << ", 1.0);\n";
      } else {
        os << "    const bool in = i < " << near << "u;\n";
        os << "    const qx::propq<double> q = qx::prop_from<double>(in ? p0 : o0, in ? p1 : o1, in ? p2 : o2, in ? p3 : o3, "
              "K0, K1, K2, K3, in ? 1.0 : -1.0, 1.0);\n";
      }
      if (overlay())
        os << "    const unsigned t = i < 4u ? 8u + i : i < 12u ? " << 24 - 4 << "u + i : " << 3 * NC + 24
           << "u + 3u * (i - 12u), d = i < 12u ? " << NC << "u : 1u;\n";
      else
        os << "    const unsigned t = " << prop0 << "u + i, d = " << NS << "u;\n";
      os << "    " << (part ? "if (i < " + std::to_string(NS) + "u) " : "") << "{\n";
      os << "      cu[t] = make_double2(q.qm, q.qp);\n      cu[t + d] = make_double2(q.q1, q.q2);\n      cu[t + 2u * d] = "
            "make_double2(q.mm, 0.0);\n    }\n  }\n";
      st.flops_per_point += (28.0 + 8 * P) * L;
    }
    sync();
  }

  // X = sum over the photons a of S of eps_a-slash C(S \ a), for the lane's
  // item of round r of level k; `off`: where the level below starts
  void vertices(int k, int r, int off, const std::string& X) {
    const int m = std::max(1, L >> k), n = (int)lv[k].size();
    for (int a = 0; a < k; ++a) {
      std::vector<int> base, ph;
      for (int t = 0; t < m; ++t) {
        const int s = k == P ? 0 : std::min(((r * L) >> k) + t, n - 1);
        uint32_t S = lv[k][s], x = S;
        for (int j = 0; j < a; ++j) x &= x - 1;
        const int p = __builtin_ctz(x);
        ph.push_back(2 * p);
        base.push_back(off + (index[k - 1][S & ~(1u << p)] << (k - 1)));
      }
      const std::string e = "qx::pol_at<" + std::to_string(2 * P) + ">(cu + " + std::to_string(pol0) + "u, " + sel(ph, k) +
                            " + ((c >> " + std::to_string(a) + ") & 1u))";
      const std::string J = k == 1 ? "u0"
                                   : get(sel(base, k) + " + ((c >> " + std::to_string(a + 1) + ") << " + std::to_string(a) +
                                         " | (c & " + std::to_string((1 << a) - 1) + "u))");
      if (a == 0)
        os << "    qx::sp4<double> " << X << " = qx::vL<double>(" << J << ", " << e << ");\n";
      else
        os << "    qx::vL_add<double>(" << X << ", " << J << ", " << e << ");\n";
      st.flops_per_point += (a ? 48.0 : 40.0) * L;
      st.n_V += L;
    }
  }

  // currents of level k over the ones of the level below
  void level(int k) {
    const int m = std::max(1, L >> k), n = (int)lv[k].size(), nr = rounds(k);
    for (int r = 0; r < nr; ++r) {
      os << "  qx::sp4<double> C" << k << "_" << r << ";\n  {\n    const unsigned c = "
         << (L >= (1 << k) ? "l" : std::to_string(r * L % (1 << k)) + "u + l") << " & " << (1 << k) - 1 << "u;\n";
      vertices(k, r, 0, "X");
      std::vector<int> at, step;
      for (int t = 0; t < m; ++t) {
        const int i = order_of(lv[k][std::min(((r * L) >> k) + t, n - 1)]);
        at.push_back(prop_at(i));
        step.push_back(prop_step(i));
      }
      for (int x : step)
        if (x != step[0]) throw std::logic_error("coop: propagator layout");
      // entries relative to the first, which fits the table's bytes
      const int at0 = at[0];
      for (int& x : at) x -= at0;
      os << "    C" << k << "_" << r << " = qx::sL<double>(X, qx::prop_at<" << step[0] << ">(cu + (" << at0 << "u + "
         << sel(at, k) << ")));\n  }\n";
      st.flops_per_point += 56.0 * L;
      st.n_S1 += L;
    }
    sync();
    for (int r = 0; r < nr; ++r) {
      // past the last item: a repeat of the last subset's, dropped
      const bool part = (r + 1) * L > items(k);
      os << "  " << (part ? "if (l < " + std::to_string(items(k) - r * L) + "u) " : "") << "qx::cur_to<" << NC << ">(cu + ("
         << r * L << "u + l), C" << k << "_" << r << ");\n";
    }
    sync();
  }

  void build() {
    prologue();
    os << "  const qx::sp4<double> u0 = qx::u_in<double>(p0, p1, p2, p3, 0, 1.0);\n";
    st.flops_per_point += 16.0 * L;
    for (int k = 1; k < P; ++k) level(k);
    // the last vertex and both spins of e-_out
    os << "  const qx::sp4<double> b0 = qx::ubar_out<double>(o0, o1, o2, o3, 0, 1.0), b1 = qx::ubar_out<double>(o0, o1, o2, "
          "o3, 1, 1.0);\n  double acc = 0.0;\n";
    st.flops_per_point += 32.0 * L;
    const int nr = std::max(1, (1 << P) / L);
    for (int r = 0; r < nr; ++r) {
      os << "  {\n    const unsigned c = " << r * L << "u + l;\n";
      vertices(P, r, 0, "F");
      os << "    const qx::cx<double> A0 = qx::dot<double>(b0, F), A1 = qx::dot<double>(b1, F);\n";
      os << "    acc += A0.r * A0.r + A0.i * A0.i + A1.r * A1.r + A1.i * A1.i;\n  }\n";
      st.flops_per_point += (60.0 + 8) * L;
      st.n_dot += 2 * L;
    }
    for (int o = 1; o < L; o <<= 1) os << "  acc += __shfl_xor(acc, " << o << ");\n";
    st.n_U = 3 + 2 * P;
    st.n_prop = NS;
  }
};

}  // namespace

// Measured, 2^20 points (99991 at 5 photons), us for 4 / 8 / 16 / 32 lanes:
// 2 photons 50 / 97 / 173 / -, 3 photons 149 / 167 / 260 / -, 4 photons 642 /
// 446 / 510 / -, 5 photons 700 / 323 / 190 / 174.  Fewer lanes need more LDS
// per wave than leaves two waves per SIMD, more lanes idle in the levels with
// few items.
int coop_lanes(const Process& pr) { return pr.P == 5 ? 32 : pr.P == 4 ? 8 : 4; }

std::string emit_coop_kernel(const Process& pr, const Variant& v, const std::string& kname, EmitStats* st) {
  Coop b(pr);
  b.build();
  if (st) *st = b.st;
  std::ostringstream os;
  os << "// generated by qedx: " << variant_tag(v, pr.n_out, pr.n_in) << "\n";
  os << "// subset currents shared by the " << b.L << " lanes of a point, one spin of e-_in\n";
  os << "#include <hip/hip_runtime.h>\n" << device_header_text() << "\n" << subset_header_text() << "\n";
  os << "extern \"C\" __global__ void __launch_bounds__(64)\n" << kname
     << "(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, double* __restrict__ out)\n{\n";
  os << "  __shared__ double2 lds[" << b.PPW * b.PT << "];\n";
  os << "  const long long pt = qx::xcd_tile() * " << b.PPW << " + threadIdx.x / " << b.L << "u;\n";
  os << "  const long long ptc = pt < N ? pt : N - 1;\n";
  os << b.os.str();
  os << "  if (pt < N && l == 0u) out[pt] = 2.0 * acc;\n}\n";
  return os.str();
}

}  // namespace qedx
