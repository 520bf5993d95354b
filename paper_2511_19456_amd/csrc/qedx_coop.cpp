// qedx_coop.cpp -- see qedx_coop.hpp.
#include "qedx_coop.hpp"

#include <algorithm>
#include <functional>
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

  // where the momenta are read: row r of the point
  std::string mrow(int r) const { return mom_lds ? "mq[" + std::to_string(64 * (r - 8)) + "u + g]" : "mom[" + std::to_string(r) + " * N + ptc]"; }
  bool ward = true;      // gradient: see reverse()
  bool mom_lds = false;  // final-state momenta of the wave's 64 points in LDS, incoming ones in pin, kin

  Coop(const Process& p, int lanes, bool grad = false) : pr(p), P(p.P), L(lanes), PPW(64 / L) {
    for (int k = 0; k <= P; ++k) {
      lv.push_back(subsets(P, k));
      index.push_back(std::vector<int>(1u << P, -1));
      for (size_t i = 0; i < lv[k].size(); ++i) index[k][lv[k][i]] = (int)i;
    }
    for (int k = 1; k < P; ++k) {
      NC = std::max(NC, items(k));
      order.insert(order.end(), lv[k].begin(), lv[k].end());
    }
    while (grad && 8 * NC < 6 * P + 4 + 4 * L) ++NC;  // the sums over the lanes
    NS = (int)order.size();
    pol0 = 4 * NC;
    prop0 = pol0 + 3 * P;
    PT = prop0 + (overlay() ? 0 : 3 * NS);
    // Lanes 0-3, 12-15 and 20-27 of a wave read 16 bytes each in one pass over
    // the 64 banks: the points' offsets keep their slots apart (12 of 16 for 8
    // lanes per point: 433 us instead of 444 with 8, 490 with 1 or 0, 2^20
    // points of 4 photons; 8 for 16 lanes: 1344 instead of 1360 us with 0, the
    // gradient of 2^18 points of 5 photons, 40 % of the conflicts)
    while (PPW > 1 && PT % 16 != (L == 8 ? 12 : L == 16 ? 8 : L % 16)) ++PT;
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
  // the lane's configuration in round r of level k
  std::string cfg(int k, int r) const {
    return "(" + (L >= (1 << k) ? std::string("l") : std::to_string(r * L % (1 << k)) + "u + l") + " & " +
           std::to_string((1 << k) - 1) + "u)";
  }
  void sync() { os << "  qx::wave_sync();\n"; }
  std::string get(const std::string& c) const {
    return "qx::cur_at<" + std::to_string(NC) + ">(cu + (" + c + "))";
  }

  // x1..x3: momentum of the lane's photon a (a lane's own load, so that no
  // photon's stays in registers for it)
  void pick_photon() {
    const int nin = pr.n_in;
    os << "    const long long pr_ = 4u * (a + (a < " << nin << "u ? 1u : 2u));\n";
    for (int mu = 1; mu < 4; ++mu) {
      const std::string m = std::to_string(mu);
      if (mom_lds)
        os << "    const double x" << m << " = a == 0u ? kin[" << m << "] : mq[64u * (unsigned)(a ? pr_ - " << 8 - mu
           << " : " << mu << ") + g];\n";
      else
        os << "    const double x" << m << " = mom[(pr_ + " << m << ") * N + ptc];\n";
    }
  }

  void prologue() {
    const int ein = pr.i_ein, eout = pr.i_eout;
    os << "  unsigned l = threadIdx.x & " << L - 1 << "u;\n";
    // opaque, so that what follows from the lane is computed where it is used
    // and not kept in registers across the loop over the groups of points
    if (mom_lds) os << "  asm volatile(\"\" : \"+v\"(l));\n";
    os << "  double2* const cu = lds + (threadIdx.x / " << L << "u) * " << PT << "u;\n";
    auto in = [&](int p, int mu) {
      return mom_lds && p < eout ? (p == ein ? "pin[" : "kin[") + std::to_string(mu) + "]" : mrow(4 * p + mu);
    };
    for (int mu = 0; mu < 4; ++mu)
      os << "  const double p" << mu << " = " << in(ein, mu) << ", o" << mu << " = " << in(eout, mu) << ";\n";
    for (int a = 0; a < P; ++a)
      for (int mu = 0; mu < 4; ++mu)
        os << "  const double k" << a << "_" << mu << " = " << (pr.photon_sign[a] < 0 ? "-" : "")
           << in(pr.photon_particle[a], mu) << ";\n";
    // polarisation vectors: item 2 a + lambda
    for (int r = 0; r * L < 2 * P; ++r) {
      os << "  {\n    const unsigned i = " << r * L << "u + l < " << 2 * P << "u ? " << r * L << "u + l : " << 2 * P - 1
         << "u;\n    const unsigned a = i >> 1;\n";
      pick_photon();
      os << "    const qx::pol3<double> e = qx::pol<double>(x1, x2, x3, (int)(i & 1u));\n";
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
      os << "  qx::sp4<double> C" << k << "_" << r << ";\n  {\n    const unsigned c = " << cfg(k, r) << ";\n";
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

  void forward() {
    prologue();
    os << "  const qx::sp4<double> u0 = qx::u_in<double>(p0, p1, p2, p3, 0, 1.0);\n";
    st.flops_per_point += 16.0 * L;
    for (int k = 1; k < P; ++k) level(k);
    // the last vertex and both spins of e-_out
    os << "  const qx::sp4<double> b0 = qx::ubar_out<double>(o0, o1, o2, o3, 0, 1.0), b1 = qx::ubar_out<double>(o0, o1, o2, "
          "o3, 1, 1.0);\n  double acc = 0.0;\n";
    st.flops_per_point += 32.0 * L;
    for (int r = 0; r < frounds(); ++r) {
      os << "  qx::sp4<double> F" << r << ";\n  qx::cx<double> A" << r << ", B" << r << ";\n";
      os << "  {\n    const unsigned c = " << r * L << "u + l;\n";
      vertices(P, r, 0, "X");
      os << "    F" << r << " = X;\n    A" << r << " = qx::dot<double>(b0, X);\n    B" << r << " = qx::dot<double>(b1, X);\n";
      os << "    " << ((r + 1) * L > (1 << P) ? "if (c < " + std::to_string(1 << P) + "u) " : "") << "acc += A" << r << ".r * A"
         << r << ".r + A" << r << ".i * A" << r << ".i + B" << r << ".r * B" << r << ".r + B" << r << ".i * B" << r
         << ".i;\n  }\n";
      st.flops_per_point += (60.0 + 8) * L;
      st.n_dot += 2 * L;
    }
    for (int o = 1; o < L; o <<= 1) os << "  acc += __shfl_xor(acc, " << o << ");\n";
    st.n_U = 3 + 2 * P;
    st.n_prop = NS;
  }
  int frounds() const { return std::max(1, (1 << P) / L); }
  bool outgoing(int a) const { return pr.photon_sign[a] < 0; }

  // Reverse sweep of log(sum |A|^2), w the adjoint of a current before its
  // propagator, written as a column like the currents (a row adjoint obeys
  // the same vertex and propagator then):
  //   w(T) = S(Q_T) sum over a not in T, lambda of eps_a-slash(lambda) w(T + a),
  // level by level downwards in LDS over the currents, which each lane keeps
  // in registers for its own items.  dS = -S dQ-slash S gives the momentum
  // gradient of a propagator from w(T) and the current C(T).
  // Through the polarisation vectors: as k turns, eps_lambda moves by
  // -(eps_lambda . dk / |k|) k/|k| and by a rotation of the two into each
  // other, which the sum over them does not see.  What is left is the
  // amplitude with k/|k| for eps_lambda, by the Ward identity minus the one
  // with (1, 0, 0, 0): the bilinear of gamma^0, 8 FMAs where the three
  // components of eps take 24 (1510 -> 1360 us for 2^18 points of 5 photons,
  // 80 -> 71 us for 20011 of 4).  Near the threshold that response is what is
  // left when the two electrons' terms cancel (their velocities, v, are all
  // that tells them apart), and the answer loses 1/v^2: there (ward = false)
  // the bilinear of k/|k| = eps_0 x eps_1 itself is taken.
  // Leaves the final-state momentum gradients through store().
  void reverse(const std::function<void()>& store) {
    // the bilinears are real parts without their factor 2: the seed carries it
    os << "  const double iS = 2.0 / acc;\n";
    for (int a = 0; a < P; ++a)
      if (outgoing(a)) {
        for (int h = 0; h < 2; ++h) os << "  double ge" << a << h << " = 0.0;\n";
        for (int mu = 0; mu < 4; ++mu) os << "  double gk" << a << mu << " = 0.0;\n";
      }
    os << "  double gh[4];\n  {\n  qx::sp4<double> wb0 = qx::zero4<double>(), wb1 = qx::zero4<double>();\n";
    sync();
    for (int r = 0; r < frounds(); ++r) {
      const bool part = (r + 1) * L > (1 << P);
      os << "  " << (part ? "if (l < " + std::to_string((1 << P) - r * L) + "u) " : "") << "{\n";
      os << "    const qx::cx<double> a = {A" << r << ".r * iS, -A" << r << ".i * iS}, b = {B" << r << ".r * iS, -B" << r
         << ".i * iS};\n    qx::axpy<double>(wb0, a, F" << r << ");\n    qx::axpy<double>(wb1, b, F" << r << ");\n";
      os << "    qx::sp4<double> w = qx::zero4<double>();\n    qx::axpy<double>(w, a, b0);\n    qx::axpy<double>(w, b, b1);\n";
      os << "    qx::cur_to<" << NC << ">(cu + (" << r * L << "u + l), qx::as_column(w));\n  }\n";
      st.flops_per_point += (4 * 32.0 + 4) * L;
    }
    // e-_out enters only here: each lane's share of its momentum gradient
    // (ubar_vjp carries the seed's factor 2)
    os << "    double h1[4];\n    qx::ubar_vjp(o0, o1, o2, o3, 0, 1.0, wb0, gh);\n    qx::ubar_vjp(o0, o1, o2, o3, 1, 1.0, wb1, h1);\n";
    os << "#pragma unroll\n    for (int m = 0; m < 4; ++m) gh[m] = 0.5 * (gh[m] + h1[m]);\n  }\n";
    st.flops_per_point += 80.0 * L;
    sync();
    for (int k = P - 1; k >= 1; --k) down(k);
    // sums over the point's lanes, through LDS: chunk of S sums at a time,
    // lane s adds the lanes' values of slot s
    std::vector<std::string> vs(6 * P + 4);
    for (int a = 0; a < P; ++a)
      if (outgoing(a)) {
        for (int h = 0; h < 2; ++h) vs[2 * a + h] = "ge" + std::to_string(a) + std::to_string(h);
        for (int mu = 0; mu < 4; ++mu) vs[2 * P + 4 * a + mu] = "gk" + std::to_string(a) + std::to_string(mu);
      }
    for (int m = 0; m < 4; ++m) vs[6 * P + m] = "gh[" + std::to_string(m) + "]";
    std::vector<int> used;
    for (size_t i = 0; i < vs.size(); ++i)
      if (!vs[i].empty()) used.push_back((int)i);
    // the last adjoints w({a}) are read before the sums take their place
    os << "  const unsigned ip = l < " << 2 * P << "u ? l : " << 2 * P - 1 << "u;\n";
    if (2 * P > L) throw std::logic_error("coop: a lane per polarisation vector");
    os << "  const qx::sp4<double> w1 = " << get("ip") << ";\n";
    sync();
    const int room = 8 * NC - (int)vs.size();  // doubles, after the results
    const int S = std::min(L, room / L);
    if (S < 1) throw std::logic_error("coop: no room for the lane sums");
    os << "  double* const rs = (double*)cu;\n  double* const ch = rs + " << vs.size() << ";\n";
    for (size_t u0 = 0; u0 < used.size(); u0 += S) {
      const int n = (int)std::min(used.size() - u0, (size_t)S);
      for (int j = 0; j < n; ++j) os << "  ch[" << j * L << "u + l] = " << vs[used[u0 + j]] << ";\n";
      sync();
      os << "  if (l < " << n << "u) {\n    double t = 0.0;\n";
      os << "#pragma unroll\n    for (unsigned j = 0; j < " << L << "u; ++j) t += ch[l * " << L << "u + ((j + l) & " << L - 1
         << "u)];\n";
      // consecutive slots but for the incoming photons' gaps
      os << "    const unsigned d = ";
      std::vector<std::pair<int, int>> runs;  // (first j, slot - j)
      for (int j = 0; j < n; ++j)
        if (runs.empty() || used[u0 + j] - j != runs.back().second) runs.push_back({j, used[u0 + j] - j});
      for (size_t q = runs.size(); q-- > 1;) os << "l >= " << runs[q].first << "u ? l + " << runs[q].second << "u : ";
      os << "l + " << runs[0].second << "u;\n    rs[d] = t;\n  }\n";
      sync();
      st.flops_per_point += (double)L * n;
    }
    // polarisation vectors to momenta, a lane each; then the photons' sums
    os << "  {\n    const unsigned i = ip, a = i >> 1;\n";
    pick_photon();
    // (zero along the z axis, where the vectors themselves have no derivative)
    os << "    const qx::pol3<double> e = qx::pol_at<" << 2 * P << ">(cu + " << pol0 << "u, i);\n";
    if (!ward)
      os << "    const double ik = qx::rsqrt(x1 * x1 + x2 * x2 + x3 * x3);\n    const qx::pol3<double> kh = {x1 * ik, x2 * ik, x3 * ik};\n";
    os << "    const double t = x1 * x1 + x2 * x2 > 0.0 ? (rs[i] + " << response("w1", "u0")
       << ") * qx::rsqrt(x1 * x1 + x2 * x2 + x3 * x3) : 0.0;\n";
    os << "    double v[3] = {t * e.e1, t * e.e2, t * e.e3};\n";
    os << "    v[0] += qx::lane_xor1(v[0]);\n    v[1] += qx::lane_xor1(v[1]);\n    v[2] += qx::lane_xor1(v[2]);\n";
    os << "    const double* const q = rs + (" << 2 * P << "u + 4u * a);\n";
    os << "    const double s = a < " << pr.n_in << "u ? 1.0 : -1.0;\n";
    os << "    const double G[4] = {s * q[0], v[0] + s * q[1], v[1] + s * q[2], v[2] + s * q[3]};\n";
    os << "    const double* const h = rs + " << 6 * P << ";\n";
    store();
    os << "  }\n";
    st.flops_per_point += 250.0 * L;
  }

  // minus the response to the spatial part of k/|k|, kh
  std::string response(const std::string& w, const std::string& C) const {
    return ward ? "qx::bil0(" + w + ", " + C + ")" : "qx_along(kh, qx::bil3(" + w + ", " + C + "))";
  }

  // whether the reverse sweep loads a step's operands during the one before:
  // 5 photons run one wave per SIMD
  bool ahead() const { return P == 5; }

  void down(int k) {
    const int m = std::max(1, L >> k), n = (int)lv[k].size(), nr = rounds(k), nj = P - k;
    const uint32_t full = (1u << P) - 1;
    auto subset = [&](int r, int t) { return lv[k][std::min(((r * L) >> k) + t, n - 1)]; };
    auto tag = [&](int r, int j) { return std::to_string(k) + "_" + std::to_string(r) + "_" + std::to_string(j); };
    // the photon of step j and the adjoints of T + a for both polarisations
    std::vector<std::vector<int>> phs(nr * nj);
    auto load = [&](int r, int j) {
      std::vector<int> base, pos, &ph = phs[r * nj + j];
      for (int t = 0; t < m; ++t) {
        const uint32_t T = subset(r, t);
        uint32_t x = full & ~T;
        for (int i = 0; i < j; ++i) x &= x - 1;
        const int p = __builtin_ctz(x);
        const uint32_t S = T | 1u << p;
        ph.push_back(2 * p);
        pos.push_back(popc(S & ((1u << p) - 1)));
        base.push_back(index[k + 1][S] << (k + 1));
      }
      const std::string g = tag(r, j);
      os << "  const unsigned ph" << g << " = " << sel(ph, k) << ";\n  qx::sp4<double> u" << g << ", v" << g << ";\n";
      os << "  {\n    const unsigned c = " << cfg(k, r) << ", ps = " << sel(pos, k) << ", lo = (1u << ps) - 1u;\n";
      os << "    const unsigned at = " << sel(base, k) << " + ((c & ~lo) << 1 | (c & lo));\n";
      os << "    u" << g << " = " << get("at") << ";\n    v" << g << " = " << get("at + (1u << ps)") << ";\n  }\n";
    };
    if (ahead()) load(0, 0);
    for (int r = 0; r < nr; ++r) {
      const bool part = (r + 1) * L > items(k);
      const std::string kr = std::to_string(k) + "_" + std::to_string(r);
      std::string C = "C" + kr;
      os << "  qx::sp4<double> W" << kr << ", G" << kr << ";\n";
      if (part) {
        // lanes past the last item repeat it and add nothing
        os << "  const qx::sp4<double> Z" << kr << " = l < " << items(k) - r * L << "u ? " << C << " : qx::zero4<double>();\n";
        C = "Z" + kr;
      }
      for (int j = 0; j < nj; ++j) {
        // one step after the other, the next one's operands under way: freely
        // interleaved they do not fit the registers
        if (!ahead()) load(r, j);
        else if (j + 1 < nj) load(r, j + 1);
        else if (r + 1 < nr) load(r + 1, 0);
        os << "  __builtin_amdgcn_sched_barrier(0);\n  {\n";
        const std::vector<int>& ph = phs[r * nj + j];
        const std::string g = tag(r, j);
        const std::string load1 = "      const double2 e1 = cu[" + std::to_string(pol0 + 1) + "u + ph" + g + "];\n";
        const std::string load0 = "      const qx::pol3<double> e0 = qx::pol_at<" + std::to_string(2 * P) + ">(cu + " +
                                  std::to_string(pol0) + "u, ph" + g + ");\n";
        if (!ward)
          os << load0 << load1
             << "      const qx::pol3<double> kh = {-e0.e3 * e1.y, e0.e3 * e1.x, e0.e1 * e1.y - e0.e2 * e1.x};\n";
        for (int h = 0; h < 2; ++h) {
          const std::string W = (h ? "v" : "u") + g;
          if (ward) os << (h ? load1 : load0);
          if (h)  // eps(1) = (-sin phi, cos phi, 0): 1344 -> 1322 us for 2^18 points of 5 photons
            os << "      qx::vL_add_flat<double>(G" << kr << ", " << W << ", e1.x, e1.y);\n";
          else
            os << "      " << (j == 0 ? "G" + kr + " = qx::vL<double>(" : "qx::vL_add<double>(G" + kr + ", ") << W << ", e0);\n";
          os << "      const double b" << h << " = " << response(W, C) << ";\n";
          st.flops_per_point += ((h ? 32.0 : 48.0) + 16) * L;
        }
        std::vector<int> seen;
        for (int t = 0; t < m; ++t) {
          const int p = ph[t] / 2;
          if (!outgoing(p) || std::find(seen.begin(), seen.end(), p) != seen.end()) continue;
          seen.push_back(p);
          bool all = true;
          for (int x : ph) all = all && x == ph[t];
          if (!all) os << "      const double m" << p << " = ph" << g << " == " << 2 * p << "u ? 1.0 : 0.0;\n";
          for (int h = 0; h < 2; ++h)
            os << "      ge" << p << h << " += " << (all ? "" : "m" + std::to_string(p) + " * ") << "b" << h << ";\n";
          st.flops_per_point += 4.0 * L;
        }
        // the sums are due here: an empty asm takes them, or the compiler
        // keeps every operand for a sum at the kernel's end
        if (!seen.empty()) {
          os << "      asm volatile(\"\" :";
          for (size_t t = 0; t < seen.size(); ++t)
            for (int h = 0; h < 2; ++h) os << (t || h ? ", " : " ") << "\"+v\"(ge" << seen[t] << h << ")";
          os << ");\n";
        }
        os << "  }\n  __builtin_amdgcn_sched_barrier(0);\n";
      }
      std::vector<int> at, step, bits;
      for (int t = 0; t < m; ++t) {
        const int i = order_of(subset(r, t));
        at.push_back(prop_at(i));
        step.push_back(prop_step(i));
        bits.push_back((int)subset(r, t));
      }
      const int at0 = at[0];
      for (int& x : at) x -= at0;
      os << "  {\n    const qx::sp4<double> w = qx::sL<double>(G" << kr << ", qx::prop_at<" << step[0] << ">(cu + (" << at0
         << "u + " << sel(at, k) << ")));\n    W" << kr << " = w;\n";
      os << "    const qx::pol3<double> b = qx::bil3(w, " << C << ");\n    const double b0 = qx::bil0(w, " << C << ");\n";
      bool same = true;
      for (int x : bits) same = same && x == bits[0];
      if (!same) os << "    const unsigned T = " << sel(bits, k) << ";\n";
      for (int a = 0; a < P; ++a) {
        if (!outgoing(a)) continue;
        bool any = false;
        for (int x : bits) any = any || ((x >> a) & 1);
        if (!any) continue;
        std::string f;
        if (!same) {
          os << "    const double m" << a << " = (T >> " << a << ") & 1u ? 1.0 : 0.0;\n";
          f = "m" + std::to_string(a) + " * ";
        }
        os << "    gk" << a << "0 -= " << f << "b0; gk" << a << "1 -= " << f << "b.e1; gk" << a << "2 -= " << f << "b.e2; gk" << a
           << "3 -= " << f << "b.e3;\n";
        os << "    asm volatile(\"\" : \"+v\"(gk" << a << "0), \"+v\"(gk" << a << "1), \"+v\"(gk" << a << "2), \"+v\"(gk" << a
           << "3));\n";
      }
      os << "  }\n";
      st.flops_per_point += (56.0 + 60 + 8 * P) * L;
    }
    sync();
    for (int r = 0; r < nr; ++r) {
      const bool part = (r + 1) * L > items(k);
      os << "  " << (part ? "if (l < " + std::to_string(items(k) - r * L) + "u) " : "") << "qx::cur_to<" << NC << ">(cu + ("
         << r * L << "u + l), W" << k << "_" << r << ");\n";
    }
    sync();
  }
};

}  // namespace

// Measured, 2^20 points (99991 at 5 photons), us for 4 / 8 / 16 / 32 lanes:
// 2 photons 50 / 97 / 173 / -, 3 photons 149 / 167 / 260 / -, 4 photons 642 /
// 446 / 510 / - (435 with the points' offsets of today), 5 photons 700 / 323 /
// 190 / 174.  Fewer lanes need more LDS
// per wave than leaves two waves per SIMD, more lanes idle in the levels with
// few items.
int coop_lanes(const Process& pr) { return pr.P == 5 ? 32 : pr.P == 4 ? 8 : 4; }

std::string emit_coop_kernel(const Process& pr, const Variant& v, const std::string& kname, EmitStats* st) {
  Coop b(pr, coop_lanes(pr));
  b.forward();
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

int coop_grad_lanes(const Process& pr) {
  return pr.P >= 4 ? 16 : 8;
}

std::string emit_coop_grad_kernel(const Process& pr, const std::string& kname, bool rambo, bool ward, EmitStats* st) {
  Coop b(pr, coop_grad_lanes(pr), true);
  b.ward = ward;
  b.mom_lds = rambo;
  if (b.overlay()) throw std::logic_error("coop: the reverse sweep reads the propagators again");
  b.forward();
  const int NF = pr.n_out + 1, L = b.L, P = pr.P;
  b.os << "  if (pt < N && l == 0u) logm2[pt] = log(2.0 * acc);\n";
  b.reverse([&]() {
    std::ostringstream& os = b.os;
    if (rambo) {
      os << "    if ((l & 1u) == 0u && l < " << 2 * P << "u && a >= " << pr.n_in << "u)\n#pragma unroll\n      for (int m = 0; m < 4; ++m) mq[64u * (4u * (a - " << pr.n_in - 1
         << "u) + m) + g] = G[m];\n";
      os << "    if (l == 0u)\n#pragma unroll\n      for (int m = 0; m < 4; ++m) mq[64u * m + g] = h[m];\n";
    } else {
      os << "    if (pt < N && (l & 1u) == 0u && l < " << 2 * P << "u && a >= " << pr.n_in << "u)\n#pragma unroll\n      for (int m = 0; m < 4; ++m) gm[(4ll * (a + 2u) + m) * N + pt] = G[m];\n";
      os << "    if (pt < N && l == 0u)\n#pragma unroll\n      for (int m = 0; m < 4; ++m) gm[(" << 4 * pr.i_eout
         << "ll + m) * N + pt] = h[m];\n";
    }
  });
  if (st) *st = b.st;
  std::ostringstream os;
  const int LDS = b.PPW * b.PT;
  if (!ward)
    os << "static __device__ __forceinline__ double qx_along(const qx::pol3<double>& k, const qx::pol3<double>& b)\n{\n"
          "  return -(k.e1 * b.e1 + k.e2 * b.e2 + k.e3 * b.e3);\n}\n";
  if (!rambo) {
    os << "extern \"C\" __global__ void __launch_bounds__(64)\n" << kname
       << "(const double* __restrict__ mom, long long N, double* __restrict__ gm, double* __restrict__ logm2)\n{\n";
    os << "  __shared__ double2 lds[" << LDS << "];\n";
    os << "  const long long pt = qx::xcd_tile() * " << b.PPW << " + threadIdx.x / " << L << "u;\n";
    os << "  const long long ptc = pt < N ? pt : N - 1;\n" << b.os.str() << "}\n";
    return os.str();
  }
  os << "extern \"C\" __global__ void __launch_bounds__(64, 2)\n" << kname
     << "(const double* __restrict__ u, double sqrt_s, long long N, double* __restrict__ logm2, double* __restrict__ grad, "
        "int tiles)\n{\n";
  os << "  __shared__ double2 lds[" << LDS << "];\n  __shared__ double mq[" << 64 * 4 * NF << "];\n";
  os << "  const long long first = qx::xcd_tile() * (long long)(tiles * " << b.PPW << ");\n";
  os << "  const bool own = threadIdx.x < (unsigned)(tiles * " << b.PPW << ");\n";
  os << "  const long long po = first + threadIdx.x < N ? first + threadIdx.x : N - 1;\n";
  os << "  if (own) {\n    double uu[" << 4 * NF << "];\n#pragma unroll\n    for (int r = 0; r < " << 4 * NF
     << "; ++r) uu[r] = u[r * N + po];\n";
  os << "    qx::RamboState<" << NF << "> S;\n    qx::rambo_forward<" << NF << ">(uu, sqrt_s, 1.0, S);\n";
  os << "#pragma unroll\n    for (int j = 0; j < " << NF << "; ++j)\n#pragma unroll\n      for (int d = 0; d < 4; ++d) mq[64 * (4 * j + "
        "d) + threadIdx.x] = S.k[j][d];\n  }\n";
  os << "  qx::wave_sync();\n  double pin[4], kin[4];\n  qx::incoming_cm(sqrt_s, 1.0, pin, kin);\n";
  os << "#pragma unroll 1\n  for (int t = 0; t < tiles; ++t) {\n";
  os << "  if (first + t * " << b.PPW << " >= N) break;\n";
  os << "  const unsigned g = (unsigned)t * " << b.PPW << "u + threadIdx.x / " << L << "u;\n  const long long pt = first + g;\n";
  os << b.os.str() << "  qx::wave_sync();\n  }\n";
  os << "  if (own && first + threadIdx.x < N) {\n    double uu[" << 4 * NF << "];\n#pragma unroll\n    for (int r = 0; r < "
     << 4 * NF << "; ++r) uu[r] = u[r * N + po];\n";
  os << "    qx::RamboState<" << NF << "> S;\n    qx::rambo_forward<" << NF << ">(uu, sqrt_s, 1.0, S);\n    double gk[" << NF
     << "][4];\n#pragma unroll\n    for (int j = 0; j < " << NF << "; ++j)\n#pragma unroll\n      for (int d = 0; d < 4; ++d) gk[j][d] = "
        "mq[64 * (4 * j + d) + threadIdx.x];\n";
  os << "    double gu[" << 4 * NF << "];\n#pragma unroll\n    for (int r = 0; r < " << 4 * NF << "; ++r) gu[r] = 0.0;\n";
  os << "    qx::rambo_vjp<" << NF << ">(uu, sqrt_s, 1.0, S, gk, gu);\n#pragma unroll\n    for (int r = 0; r < " << 4 * NF
     << "; ++r) grad[r * N + po] = gu[r];\n  }\n}\n";
  return os.str();
}

}  // namespace qedx
