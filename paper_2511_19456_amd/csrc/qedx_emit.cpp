// qedx_emit.cpp -- straight-line HIP code from the reduced QED graph.
//
// One phase-space point per lane (or 2^k lanes per point when helicity bits
// are spread over lanes).  Every compute node becomes one call of the matching
// device function of qedx_device.h; data nodes are renames (App. D: on a
// single device a data node is the identity).  The emission order groups the
// joins by photon partition so that the currents of one partition are live
// together; LLVM allocates registers for the resulting basic block.
#include "qedx_emit.hpp"
#include "qedx_pair.hpp"

#include <algorithm>
#include <array>
#include <chrono>
#include <map>
#include <set>
#include <sstream>
#include <stdexcept>

namespace qedx {

static const char* kDeviceHeaderText =
#include "qedx_device_embed.inc"
    ;

static const char* kSubsetHeaderText =
#include "qedx_subset_embed.inc"
    ;

const std::string& subset_header_text() {
  static const std::string s(kSubsetHeaderText);
  return s;
}

const std::string& device_header_text() {
  static const std::string s(kDeviceHeaderText);
  return s;
}

static int popc(uint32_t x) { return __builtin_popcount(x); }

std::string variant_tag(const Variant& v, int n_out, int n_in) {
  std::ostringstream o;
  o << "nin" << n_in << "_nout" << n_out << "_p" << v.prec << "_m" << v.mode << "_e" << v.enum_mask << "_l"
    << v.lane_mask << "_o" << v.loop_mask << "_b" << v.block << "_s" << v.split << "_j" << v.join_side << "_r"
    << v.order << "_w" << v.min_waves;
  if (v.rewrite) o << "_d" << v.rewrite;
  if (v.partial) o << "_k" << v.partial_steps << "s" << v.partial_seed;
  if (v.fixup) o << "_f" << v.fixup;
  return o.str();
}

std::string pol_lds_type(const Variant& v) {
  return v.prec == PREC_F64 || !(v.order & 64) ? "double" : "float";
}

Dag graph_for(const Process& proc, const Variant& v, double* t_build, double* t_reduce) {
  using clk = std::chrono::steady_clock;
  auto t0 = clk::now();
  Dag d = build_unreduced(proc, v.enum_mask, v.split);
  auto t1 = clk::now();
  if (v.partial) {
    // the paper's form after the first partial_steps single node reductions
    // (seeded random order), joins not split
    reduce_steps(d, v.partial_seed, v.partial_steps);
    if (t_build) *t_build = std::chrono::duration<double, std::milli>(t1 - t0).count();
    if (t_reduce) *t_reduce = std::chrono::duration<double, std::milli>(clk::now() - t1).count();
    return d;
  }
  Dag r = reduce_fixpoint(d);
  r = reduce_fixpoint(expand_joins(r, v.join_side));
  r = compact(r);
  if (v.rewrite == 1) r = distribute(r);
  auto t2 = clk::now();
  if (t_build) *t_build = std::chrono::duration<double, std::milli>(t1 - t0).count();
  if (t_reduce) *t_reduce = std::chrono::duration<double, std::milli>(t2 - t1).count();
  return r;
}

namespace {

struct Emitter {
  const Dag& d;
  const Variant& v;
  const Process& pr;
  std::ostringstream os;
  std::vector<char> done;
  std::set<uint32_t> kdone;
  std::set<std::pair<int, uint32_t>> qdone;
  std::map<int, int> acc_of_sum;  // Sum node -> accumulator index
  EmitStats st;
  std::string T;
  std::string ind = "  ";
  // Partition loop: one block for the canonical partition (photons 0..split-1
  // on the e-_in side) inside a run-time loop over all partitions; photon
  // slot a of iteration `it` is particle slot_tab[it][a], loaded per iteration.
  bool slot = false;
  std::string slot_tab;

  int slot_of(int particle) const {
    for (int a = 0; a < pr.P; ++a)
      if (pr.photon_particle[a] == particle) return a;
    return -1;
  }

  Emitter(const Dag& d_, const Variant& v_) : d(d_), v(v_), pr(d_.proc), done(d_.nodes.size(), 0) {
    T = v.prec == PREC_F64 ? "double" : "float";
    d1 = v.prec != PREC_F64 && !(v.order & 64);
    PT = pol_lds_type(v);
  }

  // FP32C: the first vertex and propagator next to each external electron
  // (U -> V -> S1) are evaluated in FP64 and rounded once.  There
  // (Qslash + m) eps-slash u(p) = eps-slash kslash u + 2 (eps.p) u for
  // Q = p - k, so with eps.p ~ 0 and a soft k the product cancels by
  // ~2E/k; in FP32 that cancellation costs as many digits (likewise
  // ubar(p') eps-slash (p'-slash + kslash + m) on the other side).  Nodes with an
  // FP64 copy are named <name>_d.
  bool d1 = false;
  std::string PT;  // element type of the per-lane polarisation LDS
  std::set<int> has_d;
  std::set<std::pair<int, uint32_t>> qdone_d;

  int producer(int i) const {
    const Node& n = d.nodes[i];
    return n.kind == Kind::Data ? n.in[0] : i;
  }
  std::string name(int i) const {
    auto a = alias.find(producer(i));
    return a != alias.end() ? a->second : "n" + std::to_string(producer(i));
  }
  // LDS staging of the held side of each partition block (order flag 16):
  // the held currents are stored to per-lane LDS slots once and read back,
  // through an address the compiler cannot see through, for every group of
  // kTile streamed currents -- register pressure is then the accumulators,
  // one tile and one held current.
  std::map<int, std::string> alias;
  bool batch_mom = false;  // order flag 8192: block momenta loaded together (see block_momenta)
  bool stage() const { return (v.order & 16) != 0; }
  int lds_slots = 0;
  // partition slot loop: photon polarisation vectors computed once per point
  // (and helicity-loop iteration) before the loop, kept in per-lane LDS and
  // read by slot inside it, instead of once per partition
  bool pol_lds = false;
  static constexpr int kTile = 4;
  // One-photon current cache (order flag 256, per-point FP64 slot loops):
  // the two lanes of a point first compute, for every photon, its
  // polarisation vector and its one-photon currents on both sides,
  // S(Q) eps-slash u and ubar eps-slash S(Q), into per-point LDS; the
  // partition loop, split between the two lanes, reads them there instead of
  // recomputing them in every partition (each photon's one-photon current
  // is otherwise rebuilt once per partition that puts the photon first on a
  // side).  BP = points per workgroup.
  bool cur_cache = false;
  int BP = 0, CL = 1;  // points per workgroup, lanes per point
  bool k_lds = false;  // the signed photon momenta cached too (where LDS allows)
  bool row_only = false;  // order flag 1024: only the e-_in side's currents cached
  // Shared e-_in side (order flag 2048; SUM kernels whose one lane bit is
  // the e-_out spin and whose graph enumerates the e-_in spin): both lanes of
  // a point would build the same e-_in-side currents for both e-_in spins.
  // Instead each lane builds them for one e-_in spin (its lane bit) and takes
  // the other spin's leaves from its partner lane.  Lane 1 thereby swaps the
  // e-_in labels of all its accumulators, which leaves sum |A|^2 unchanged.
  bool coop = false;
  std::map<std::pair<int, int>, int> v_of;  // (photon state, current) -> V node
  std::map<int, int> s1_of;                 // current -> S1 node
  int u_ein0 = -1;                          // U node of e-_in with spin 0
  bool ein1(int x) const {  // an e-_in-side value of e-_in spin 1
    const Node& n = d.nodes[x];
    const uint32_t b = 1u << pr.i_ein;
    return coop && n.side == 0 && (n.kind == Kind::V || n.kind == Kind::S1) && (n.cfg_dep & b) && (n.cfg & b);
  }
  void build_twins() {
    for (size_t i = 0; i < d.nodes.size(); ++i) {
      const Node& n = d.nodes[i];
      if (n.kind == Kind::V) v_of[{producer(n.in[0]), producer(n.in[1])}] = (int)i;
      if (n.kind == Kind::S1) s1_of[producer(n.in[0])] = (int)i;
      if (n.kind == Kind::U && n.particle == pr.i_ein && n.hel == 0) u_ein0 = (int)i;
    }
    if (u_ein0 < 0) throw std::invalid_argument("shared e-_in side: no enumerated e-_in spin");
  }
  // the same value with e-_in spin 0
  int twin(int x) const {
    x = producer(x);
    const Node& n = d.nodes[x];
    if (n.kind == Kind::U) return n.particle == pr.i_ein ? u_ein0 : x;
    if (n.kind == Kind::V) return v_of.at({producer(n.in[0]), twin(n.in[1])});
    if (n.kind == Kind::S1) return s1_of.at(twin(n.in[0]));
    throw std::logic_error("shared e-_in side: unexpected node kind");
  }

  // e-_in-side one-photon currents of a helicity-sum kernel (order flag
  // 4096, with the shared e-_in side): every partition block that puts a
  // photon first on the e-_in side rebuilt S(Q) eps-slash u for each of its
  // polarisation states; they are computed once per point (and loop
  // iteration) into per-lane LDS, [slot][8 words][block], and read there.
  bool r1_cache = false;
  std::map<int, int> r1_slot;  // S1 node -> LDS slot
  std::string r1_ref(int slot, int w) const {
    return "qx_r1[" + std::to_string((8 * slot + w) * v.block) + " + threadIdx.x]";
  }
  void r1_collect() {
    for (size_t i = 0; i < d.nodes.size(); ++i) {
      const Node& n = d.nodes[i];
      if (n.kind == Kind::S1 && n.side == 0 && popc(n.mask) == 1 && !ein1((int)i) && !n.out.empty())
        r1_slot[(int)i] = (int)r1_slot.size();
    }
  }
  void emit_r1_cache() {
    os << ind << "{\n";
    std::string o = ind;
    ind += "  ";
    block_momenta();
    std::fill(done.begin(), done.end(), 0);
    kdone.clear();
    qdone.clear();
    const bool was = r1_cache;
    r1_cache = false;  // compute them here
    for (auto& kv : r1_slot) {
      emit(kv.first);
      for (int k = 0; k < 4; ++k)
        os << ind << r1_ref(kv.second, 2 * k) << " = " << name(kv.first) << ".c[" << k << "].r; "
           << r1_ref(kv.second, 2 * k + 1) << " = " << name(kv.first) << ".c[" << k << "].i;\n";
    }
    r1_cache = was;
    std::fill(done.begin(), done.end(), 0);
    kdone.clear();
    qdone.clear();
    ind = o;
    os << ind << "}\n";
  }

  // a device-function body of the persistent batch kernel: the cache is the
  // wave's own LDS region (BP = points per wave), tpt and sub are arguments,
  // and the wave synchronises only itself
  bool body_mode = false;
  void wave_sync() {
    os << ind << "__builtin_amdgcn_fence(__ATOMIC_RELEASE, \"wavefront\"); __builtin_amdgcn_wave_barrier(); "
       << "__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, \"wavefront\");\n";
  }
  std::string ix_tab;  // photon index of every slot: [iteration][P]
  std::string cache_k(const std::string& ix, int mu) const {
    return "qx_k[(4 * " + ix + " + " + std::to_string(mu) + ") * " + std::to_string(BP) + " + tpt]";
  }
  std::string cache_pol(const std::string& ix, int c) const {
    return "qx_pol[(3 * " + ix + " + " + std::to_string(c) + ") * " + std::to_string(BP) + " + tpt]";
  }
  std::string cache_cur(int side, const std::string& ix, int w) const {
    return "qx_cur[(" + std::to_string(side * pr.P * 8 + w) + " + 8 * " + ix + ") * " + std::to_string(BP) + " + tpt]";
  }

  void emitK(uint32_t mask) {
    if (kdone.count(mask)) return;
    int lo = __builtin_ctz(mask);
    uint32_t rest = mask & (mask - 1);
    std::string km = "K" + std::to_string(mask);
    if (rest == 0 && slot && k_lds) {
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double " << km << "_" << mu << " = " << cache_k("ix" + std::to_string(lo), mu) << ";\n";
    } else if (rest == 0 && slot) {
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double " << km << "_" << mu << " = sg" << lo << " * k" << lo << "_" << mu << ";\n";
      st.flops_per_point += 4;
    } else if (rest == 0) {
      int part = pr.photon_particle[lo];
      const char* sg = pr.photon_sign[lo] > 0 ? "" : "-";
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double " << km << "_" << mu << " = " << sg << "m" << part << "_" << mu << ";\n";
    } else {
      emitK(rest);
      emitK(1u << lo);
      std::string kr = "K" + std::to_string(rest), kl = "K" + std::to_string(1u << lo);
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double " << km << "_" << mu << " = " << kr << "_" << mu << " + " << kl << "_" << mu
           << ";\n";
      st.flops_per_point += 4;
    }
    kdone.insert(mask);
  }

  std::string qname(int side, uint32_t mask) const {
    return std::string(side == 0 ? "qL" : "qR") + std::to_string(mask);
  }

  void emitQ(int side, uint32_t mask) {
    if (qdone.count({side, mask})) return;
    emitK(mask);
    int pp = side == 0 ? pr.i_ein : pr.i_eout;
    std::string km = "K" + std::to_string(mask);
    os << ind << "const qx::propq<" << T << "> " << qname(side, mask) << " = qx::prop_from<" << T << ">(m" << pp
       << "_0, m" << pp << "_1, m" << pp << "_2, m" << pp << "_3, " << km << "_0, " << km << "_1, " << km << "_2, "
       << km << "_3, " << (side == 0 ? "1.0" : "-1.0") << ", 1.0);\n";
    if (!qdone_d.count({side, mask})) {
      st.flops_per_point += 28;
      ++st.n_prop;
    }
    qdone.insert({side, mask});
  }

  // FP64 propagator coefficients (for the FP32C first-step currents)
  void emitQd(int side, uint32_t mask) {
    if (qdone_d.count({side, mask})) return;
    emitK(mask);
    int pp = side == 0 ? pr.i_ein : pr.i_eout;
    std::string km = "K" + std::to_string(mask);
    os << ind << "const qx::propq<double> " << qname(side, mask) << "_d = qx::prop_from<double>(m" << pp << "_0, m"
       << pp << "_1, m" << pp << "_2, m" << pp << "_3, " << km << "_0, " << km << "_1, " << km << "_2, " << km
       << "_3, " << (side == 0 ? "1.0" : "-1.0") << ", 1.0);\n";
    if (!qdone.count({side, mask})) {
      st.flops_per_point += 28;
      ++st.n_prop;
    }
    qdone_d.insert({side, mask});
  }
  std::string name_d(int i) const { return "n" + std::to_string(producer(i)) + "_d"; }

  std::string hel_expr(const Node& u) const {
    if (coop && u.particle == pr.i_ein) return "(int)((hc >> " + std::to_string(pr.i_eout) + ") & 1u)";
    if (u.hel >= 0) return std::to_string((int)u.hel);
    if (slot && slot_of(u.particle) >= 0) return "hb" + std::to_string(slot_of(u.particle));
    return "(int)((hc >> " + std::to_string(u.particle) + ") & 1u)";
  }

  bool local() const { return (v.order & 4) != 0 && !slot; }
  bool loop_local() const { return (v.order & 32) != 0 && v.loop_mask != 0 && !local() && !slot; }

  // scheduling fence: keeps LLVM's machine scheduler from moving work across
  void fence(int level) {
    if (v.order & level) os << ind << "__builtin_amdgcn_sched_barrier(0);\n";
  }

  void emit(int i) {
    int c = producer(i);
    if (done[c]) return;
    const Node& n = d.nodes[c];
    if (r1_cache && r1_slot.count(c)) {
      os << ind << "const qx::sp4<" << T << "> n" << c << " = {{";
      for (int k = 0; k < 4; ++k)
        os << (k ? ", " : "") << "{" << r1_ref(r1_slot.at(c), 2 * k) << ", " << r1_ref(r1_slot.at(c), 2 * k + 1) << "}";
      os << "}};\n";
      done[c] = 1;
      return;
    }
    if (ein1(c)) {
      // built by the partner lane as its spin-0 twin
      const int t = twin(c);
      emit(t);
      os << ind << "const qx::sp4<" << T << "> n" << c << " = qx::lane_xor1(" << name(t) << ");\n";
      done[c] = 1;
      return;
    }
    if (cur_cache && n.kind == Kind::S1 && popc(n.mask) == 1 && (n.side == 0 || !row_only)) {
      // a one-photon current: read from the per-point cache
      const std::string ix = "ix" + std::to_string(__builtin_ctz(n.mask));
      os << ind << "const qx::sp4<" << T << "> n" << c << " = {{";
      for (int k = 0; k < 4; ++k)
        os << (k ? ", " : "") << "{" << cache_cur(n.side, ix, 2 * k) << ", " << cache_cur(n.side, ix, 2 * k + 1) << "}";
      os << "}};\n";
      done[c] = 1;
      return;
    }
    for (int p : n.in) emit(p);
    std::string nm = "n" + std::to_string(c);
    switch (n.kind) {
      case Kind::Entry: break;
      case Kind::U: {
        int p = n.particle;
        std::string m = "m" + std::to_string(p) + "_";
        // with d1 the state is built in FP64 (name_d) and rounded for the FP32 graph
        const std::string TU = d1 ? "double" : T;
        const std::string nu = d1 ? nm + "_d" : nm;
        if (p == pr.i_ein || p == pr.i_eout) {
          os << ind << "const qx::sp4<" << TU << "> " << nu << " = qx::" << (p == pr.i_ein ? "u_in" : "ubar_out") << "<"
             << TU << ">(" << m << "0, " << m << "1, " << m << "2, " << m << "3, " << hel_expr(n) << ", 1.0);\n";
          if (d1) os << ind << "const qx::sp4<float> " << nm << " = qx::to_f(" << nu << ");\n";
        } else if (cur_cache) {
          // polarisation from the per-point cache, in the graph's type (the
          // FP64 first steps that need it in FP64 are cached themselves)
          os << ind << "const qx::pol3<" << T << "> " << nm << " = {";
          for (int c = 0; c < 3; ++c) os << (c ? ", " : "") << cache_pol("ix" + std::to_string(slot_of(p)), c);
          os << "};\n";
          st.flops_per_point += 16;
          ++st.n_U;
          break;
        } else if (slot && pol_lds) {
          std::string sp = "sp" + std::to_string(slot_of(p));
          os << ind << "const qx::pol3<" << TU << "> " << nu << " = {";
          for (int c = 0; c < 3; ++c)
            os << (c ? ", " : "") << (PT != TU ? "(" + TU + ")" : std::string())
               << "qx_pol[(3 * " << sp << " + " << c << ") * " << v.block << " + threadIdx.x]";
          os << "};\n";
          if (d1) os << ind << "const qx::pol3<float> " << nm << " = qx::to_f(" << nu << ");\n";
        } else {
          if (slot) m = "k" + std::to_string(slot_of(p)) + "_";
          os << ind << "const qx::pol3<" << TU << "> " << nu << " = qx::pol<" << TU << ">(" << m << "1, " << m << "2, "
             << m << "3, " << hel_expr(n) << ");\n";
          if (d1) os << ind << "const qx::pol3<float> " << nm << " = qx::to_f(" << nu << ");\n";
        }
        if (d1) has_d.insert(c);
        st.flops_per_point += 16;
        ++st.n_U;
        break;
      }
      case Kind::V: {
        const Node& ph = d.nodes[producer(n.in[0])];
        bool y = ph.hel == 1;
        const Node& cur = d.nodes[producer(n.in[1])];
        if (d1 && cur.kind == Kind::U && has_d.count(producer(n.in[1])) && has_d.count(producer(n.in[0]))) {
          // first vertex next to an external electron: FP64, rounded once
          os << ind << "const qx::sp4<double> " << nm << "_d = qx::v" << (n.side == 0 ? "L" : "R") << (y ? "_y" : "")
             << "<double>(" << name_d(n.in[1]) << ", " << name_d(n.in[0]) << ");\n";
          os << ind << "const qx::sp4<float> " << nm << " = qx::to_f(" << nm << "_d);\n";
          has_d.insert(c);
        } else {
          os << ind << "const qx::sp4<" << T << "> " << nm << " = qx::v" << (n.side == 0 ? "L" : "R")
             << (y ? "_y" : "") << "<" << T << ">(" << name(n.in[1]) << ", " << name(n.in[0]) << ");\n";
        }
        st.flops_per_point += y ? 24 : 40;
        ++st.n_V;
        break;
      }
      case Kind::S1: {
        if (d1 && d.nodes[producer(n.in[0])].kind == Kind::V && has_d.count(producer(n.in[0]))) {
          // propagator after the first vertex: FP64 on the FP64 current, rounded once
          emitQd(n.side, n.mask);
          os << ind << "const qx::sp4<double> " << nm << "_d = qx::s" << (n.side == 0 ? "L" : "R") << "<double>("
             << name_d(n.in[0]) << ", " << qname(n.side, n.mask) << "_d);\n";
          os << ind << "const qx::sp4<float> " << nm << " = qx::to_f(" << nm << "_d);\n";
          has_d.insert(c);
        } else {
          emitQ(n.side, n.mask);
          os << ind << "const qx::sp4<" << T << "> " << nm << " = qx::s" << (n.side == 0 ? "L" : "R") << "<" << T
             << ">(" << name(n.in[0]) << ", " << qname(n.side, n.mask) << ");\n";
        }
        st.flops_per_point += 56;
        ++st.n_S1;
        break;
      }
      case Kind::Add: {
        std::string e = name(n.in[0]);
        for (size_t t = 1; t < n.in.size(); ++t)
          e = "qx::add4<" + T + ">(" + e + ", " + name(n.in[t]) + ")";
        os << ind << "const qx::sp4<" << T << "> " << nm << " = " << e << ";\n";
        st.flops_per_point += 8.0 * (double)(n.in.size() - 1);
        break;
      }
      case Kind::Dot:
      case Kind::Sum:
      case Kind::HelSum:
      case Kind::S2:
        throw std::logic_error("emit(): joins and sums are emitted by the caller");
      default: break;
    }
    done[c] = 1;
    if (n.kind != Kind::Entry) fence(2);
  }

  // the two operands of a Dot: (column current J, row current B)
  std::pair<int, int> dot_ops(const Node& n) const {
    int a = n.in[0], b = n.in[1];
    if (d.nodes[producer(a)].side != 0) std::swap(a, b);
    return {a, b};
  }

  void emit_dot(int k) {
    const Node& n = d.nodes[k];
    auto ops = dot_ops(n);
    int sum = n.out.empty() ? -1 : d.nodes[n.out[0]].out[0];  // Dot -> Data -> Sum
    int acc = acc_of_sum.at(sum);
    std::string B = name(ops.second);
    if (n.kind == Kind::S2) {
      // join of the paper's form (graphs that were not split): the row
      // current is propagated here, Jbar S(Q) J
      uint32_t mb = d.nodes[producer(ops.second)].mask;
      emitQ(1, mb);
      B = "qx::sR<" + T + ">(" + B + ", " + qname(1, mb) + ")";
      st.flops_per_point += 56;
    }
    if (v.prec == PREC_F64) {
      os << ind << "qx::dot_acc<double>(A" << acc << ", " << B << ", " << name(ops.first) << ");\n";
      st.flops_per_point += 32;
    } else {
      // a join of two FP64 first-step currents (one photon on each side):
      // the dot in FP64 too, the diagram value rounded once
      std::string x = "qx::dot<float>(" + B + ", " + name(ops.first) + ")";
      if (n.kind == Kind::Dot && has_d.count(producer(ops.second)) && has_d.count(producer(ops.first)))
        x = "qx::to_f(qx::dot<double>(" + name_d(ops.second) + ", " + name_d(ops.first) + "))";
      if (abs_sum) {
        os << ind << "{ const qx::cx<float> x_ = " << x << "; qx::comp_acc<float>(A" << acc << ", C" << acc
           << ", x_); S" << acc << " = fmaf(x_.r, x_.r, fmaf(x_.i, x_.i, S" << acc << ")); }\n";
        st.flops_per_point += 30 + 14 + 2;
      } else {
        os << ind << "qx::comp_acc<float>(A" << acc << ", C" << acc << ", " << x << ");\n";
        st.flops_per_point += 30 + 14;
      }
    }
    ++st.n_dot;
    fence(2);
  }

  // FP32C per-point fix-up: sum |diagram value| beside the compensated sum
  // and raise `fixflag` (declared by the kernel) on cancellation
  bool abs_sum = false;

  std::vector<int> sum_nodes() const {
    std::vector<int> sums;
    for (size_t i = 0; i < d.nodes.size(); ++i)
      if (d.nodes[i].kind == Kind::Sum) sums.push_back((int)i);
    return sums;
  }

  // Dots grouped by the photon set on the e-_in side (one group per
  // partition), and an order of the groups in which consecutive partitions
  // share as many photons as possible.
  void partitions(std::map<uint32_t, std::vector<int>>& part, std::vector<uint32_t>& order) const {
    for (size_t i = 0; i < d.nodes.size(); ++i)
      if (d.nodes[i].kind == Kind::Dot || d.nodes[i].kind == Kind::S2) {
        auto ops = dot_ops(d.nodes[i]);
        part[d.nodes[producer(ops.first)].mask].push_back((int)i);
      }
    std::vector<uint32_t> keys;
    for (auto& kv : part) keys.push_back(kv.first);
    std::vector<char> used(keys.size(), 0);
    uint32_t cur = keys.empty() ? 0 : keys[0];
    for (size_t t = 0; t < keys.size(); ++t) {
      int best = -1, bscore = -1;
      for (size_t q = 0; q < keys.size(); ++q) {
        if (used[q]) continue;
        int sc = t == 0 ? (q == 0 ? 1 : 0) : popc(keys[q] & cur);
        if (sc > bscore) {
          bscore = sc;
          best = (int)q;
        }
      }
      used[best] = 1;
      cur = keys[best];
      order.push_back(cur);
    }
  }

  // Partition-local block: momenta reloaded through a value the compiler
  // cannot see through, so nothing computed here is merged with (and kept
  // live from) another partition's block; a uniform branch on an opaque flag
  // puts the block in its own basic block, so instruction selection
  // schedules it on its own.
  std::string open_block() {
    std::string outer = ind;
    os << ind << "{\n" << ind << "  int live = 1;\n" << ind << "  asm volatile(\"\" : \"+s\"(live));\n" << ind
       << "  if (live) {\n";
    ind += "    ";
    block_momenta();
    std::fill(done.begin(), done.end(), 0);
    kdone.clear();
    qdone.clear();
    qdone_d.clear();
    has_d.clear();
    return outer;
  }
  void close_block(const std::string& outer) {
    ind = outer;
    os << ind << "  }\n" << ind << "}\n";
  }

  void forward_block(uint32_t key, const std::vector<int>& dk) {
    fence(1);
    os << ind << "// photons " << key << " | " << (((1u << pr.P) - 1) & ~key) << " on the e-_in | e-_out side\n";
    std::string outer;
    if (local()) outer = open_block();
    forward_block_inner(key, dk);
    if (local()) close_block(outer);
  }

  // opaque per-use LDS index (the base stays visible, so accesses stay ds_*)
  std::string lds_index(int slot) const {
    return "int ix = " + std::to_string(slot * 8 * v.block) + " + (int)threadIdx.x; asm volatile(\"\" : \"+v\"(ix));";
  }

  void staged_block(const std::vector<int>& dk, const std::set<int>& hold, const std::set<int>& stream, bool holdB) {
    std::vector<int> hv(hold.begin(), hold.end()), sv(stream.begin(), stream.end());
    lds_slots = std::max(lds_slots, (int)hv.size());
    for (size_t k = 0; k < hv.size(); ++k) {
      emit(hv[k]);
      os << ind << "{ " << lds_index((int)k) << " qx::lds_put<" << T << ">(qx_lds + ix, " << v.block << ", "
         << name(hv[k]) << "); }\n";
    }
    std::map<std::pair<int, int>, std::vector<int>> dots;  // (held, streamed) -> Dot nodes
    for (int k : dk) {
      auto ops = dot_ops(d.nodes[k]);
      int J = producer(ops.first), B = producer(ops.second);
      dots[holdB ? std::make_pair(B, J) : std::make_pair(J, B)].push_back(k);
    }
    for (size_t t0 = 0; t0 < sv.size(); t0 += kTile) {
      size_t t1 = std::min(sv.size(), t0 + kTile);
      for (size_t t = t0; t < t1; ++t) emit(sv[t]);
      for (size_t k = 0; k < hv.size(); ++k) {
        bool any = false;
        for (size_t t = t0; t < t1 && !any; ++t) any = dots.count({hv[k], sv[t]}) > 0;
        if (!any) continue;
        std::string tmp = "h" + std::to_string(hv[k]) + "_" + std::to_string(t0);
        os << ind << "{\n";
        std::string outer = ind;
        ind += "  ";
        os << ind << lds_index((int)k) << "\n";
        os << ind << "const qx::sp4<" << T << "> " << tmp << " = qx::lds_get<" << T << ">(qx_lds + ix, " << v.block
           << ");\n";
        alias[hv[k]] = tmp;
        for (size_t t = t0; t < t1; ++t) {
          auto it = dots.find({hv[k], sv[t]});
          if (it == dots.end()) continue;
          for (int dkk : it->second) emit_dot(dkk);
        }
        alias.erase(hv[k]);
        ind = outer;
        os << ind << "}\n";
      }
    }
  }

  void forward_block_inner(uint32_t key, const std::vector<int>& dk) {
    (void)key;
    std::set<int> Bs, Js;
    for (int k : dk) {
      auto ops = dot_ops(d.nodes[k]);
      Js.insert(producer(ops.first));
      Bs.insert(producer(ops.second));
    }
    bool holdB = Bs.size() <= Js.size();
    const std::set<int>& hold = holdB ? Bs : Js;
    const std::set<int>& stream = holdB ? Js : Bs;
    if (stage()) {
      staged_block(dk, hold, stream, holdB);
      return;
    }
    for (int h : hold) emit(h);
    auto stream_one = [&](int s) {
      emit(s);
      for (int k : dk) {
        auto ops = dot_ops(d.nodes[k]);
        int sp = producer(holdB ? ops.first : ops.second);
        if (sp == s) emit_dot(k);
      }
    };
    // with the shared e-_in side each spin-1 leaf follows its spin-0 twin
    std::map<int, int> after;
    if (coop && !holdB)
      for (int s : stream)
        if (ein1(s) && stream.count(twin(s))) after[twin(s)] = s;
    for (int s : stream) {
      if (coop && !holdB && ein1(s) && stream.count(twin(s))) continue;
      stream_one(s);
      auto a = after.find(s);
      if (a != after.end()) stream_one(a->second);
    }
  }

  // The partitions of the photons into the two sides of the joins, in the
  // slot order used by slot_loop: iteration t puts photons subsets[t] on the
  // e-_in side; returns the table of particle indices [NIT][P].
  std::vector<int> slot_table() const {
    const int P = pr.P, j = d.split;
    std::vector<int> tab;
    for (uint32_t m = 0; m < (1u << P); ++m) {
      if (popc(m) != j) continue;
      for (int a = 0; a < P; ++a)
        if ((m >> a) & 1) tab.push_back(pr.photon_particle[a]);
      for (int a = 0; a < P; ++a)
        if (!((m >> a) & 1)) tab.push_back(pr.photon_particle[a]);
    }
    return tab;
  }

  void emit_slot_table() {
    std::vector<int> tab = slot_table();
    os << "__constant__ int " << slot_tab << "[" << tab.size() << "] = {";
    for (size_t i = 0; i < tab.size(); ++i) os << (i ? ", " : "") << tab[i];
    os << "};\n";
    if (cur_cache) {
      os << "__constant__ int " << ix_tab << "[" << tab.size() << "] = {";
      for (size_t i = 0; i < tab.size(); ++i) os << (i ? ", " : "") << slot_of(tab[i]);
      os << "};\n";
    }
  }

  void slot_loop(std::map<uint32_t, std::vector<int>>& part) {
    const int P = pr.P;
    const uint32_t key = (1u << d.split) - 1;
    const int nit = (int)(slot_table().size() / P);
    if (!part.count(key)) throw std::logic_error("canonical partition missing");
    for (int p : {pr.i_ein, pr.i_eout})
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double m" << p << "_" << mu << " = mom[" << (4 * p + mu) << " * N + ptc];\n";
    if (pol_lds && !cur_cache)
      for (int a = 0; a < P; ++a) {
        int pp = pr.photon_particle[a];
        os << ind << "{ const qx::pol3<" << PT << "> e_ = qx::pol<" << PT << ">(mom[" << (4 * pp + 1) << " * N + ptc], mom["
           << (4 * pp + 2) << " * N + ptc], mom[" << (4 * pp + 3) << " * N + ptc], (int)((hc >> " << pp << ") & 1u));";
        for (int c = 0; c < 3; ++c)
          os << " qx_pol[" << (3 * pp + c) * v.block << " + threadIdx.x] = e_.e" << (c + 1) << ";";
        os << " }\n";
      }
    double pre = 0.0;  // FLOPs per lane before the loop
    if (cur_cache) {
      // photons sub, sub + 2, ... of the point: polarisation vector and the
      // two one-photon currents into the per-point cache (photon index a is
      // particle a + 1 for the n_in incoming photons, a + 2 after e-_out)
      const int ein = pr.i_ein, eout = pr.i_eout, nin = eout - 1;
      auto mref = [&](int p) {
        std::string m = "m" + std::to_string(p) + "_";
        return m + "0, " + m + "1, " + m + "2, " + m + "3";
      };
      if (body_mode)
        wave_sync();  // the previous tile's reads of the region come first
      else
        os << ind << "const int tpt = (int)(threadIdx.x >> " << __builtin_ctz(CL) << ");\n";
      os << ind << "const int q_ = (int)(sub & " << CL - 1 << "u);\n";
      os << ind << "{\n";
      os << ind << "  const qx::sp4<double> ue_ = qx::u_in<double>(" << mref(ein) << ", (int)((hc >> " << ein
         << ") & 1u), 1.0);\n";
      if (!row_only)
        os << ind << "  const qx::sp4<double> ub_ = qx::ubar_out<double>(" << mref(eout) << ", (int)((hc >> " << eout
           << ") & 1u), 1.0);\n";
      os << ind << "  #pragma unroll\n" << ind << "  for (int j = 0; j < " << (P + CL - 1) / CL << "; ++j) {\n";
      os << ind << "    const int a = " << CL << " * j + q_;\n";
      os << ind << "    if (a < " << P << ") {\n";
      os << ind << "      const int pp = a + (a < " << nin << " ? 1 : 2);\n";
      os << ind << "      const double s_ = a < " << nin << " ? 1.0 : -1.0;\n";
      os << ind << "      double k_[4];\n";
      os << ind << "      for (int mu = 0; mu < 4; ++mu) k_[mu] = mom[(4 * pp + mu) * N + ptc];\n";
      os << ind << "      const qx::pol3<double> e_ = qx::pol<double>(k_[1], k_[2], k_[3], (int)((hc >> pp) & 1u));\n";
      for (int c = 0; c < 3; ++c) os << ind << "      " << cache_pol("a", c) << " = (" << T << ")e_.e" << (c + 1) << ";\n";
      if (k_lds)
        for (int mu = 0; mu < 4; ++mu) os << ind << "      " << cache_k("a", mu) << " = s_ * k_[" << mu << "];\n";
      os << ind << "      const qx::sp4<double> r_ = qx::sL<double>(qx::vL<double>(ue_, e_), qx::prop_from<double>("
         << mref(ein) << ", s_ * k_[0], s_ * k_[1], s_ * k_[2], s_ * k_[3], 1.0, 1.0));\n";
      if (!row_only)
        os << ind << "      const qx::sp4<double> c_ = qx::sR<double>(qx::vR<double>(ub_, e_), qx::prop_from<double>("
           << mref(eout) << ", s_ * k_[0], s_ * k_[1], s_ * k_[2], s_ * k_[3], -1.0, 1.0));\n";
      for (int side = 0; side < (row_only ? 1 : 2); ++side)
        for (int k = 0; k < 4; ++k)
          os << ind << "      " << cache_cur(side, "a", 2 * k) << " = (" << T << ")" << (side ? "c_" : "r_") << ".c[" << k
             << "].r; " << cache_cur(side, "a", 2 * k + 1) << " = (" << T << ")" << (side ? "c_" : "r_") << ".c[" << k
             << "].i;\n";
      os << ind << "    }\n" << ind << "  }\n" << ind << "}\n";
      if (body_mode)
        wave_sync();
      else
        os << ind << "__syncthreads();\n";
      pre = (row_only ? 16 : 2 * 16) + (P + CL - 1) / CL * (16 + 4 + (row_only ? 1 : 2) * (40 + 28 + 56));
    }
    std::string outer = ind;
    if (!cur_cache) {
      os << ind << "#pragma unroll 1\n" << ind << "for (int it = 0; it < " << nit << "; ++it) {\n";
      ind += "  ";
      for (int a = 0; a < P; ++a) {
        os << ind << "const int sp" << a << " = " << slot_tab << "[it * " << P << " + " << a << "];\n";
        os << ind << "const double sg" << a << " = sp" << a << " < " << pr.i_eout << " ? 1.0 : -1.0;\n";
        os << ind << "const int hb" << a << " = (int)((hc >> sp" << a << ") & 1u);\n";
        for (int mu = 0; mu < 4; ++mu)
          os << ind << "const double k" << a << "_" << mu << " = mom[(4 * sp" << a << " + " << mu << ") * N + ptc];\n";
      }
    } else {
      // lane q of a point takes partitions CL i2 + q: the loop index stays
      // uniform, so the table entries are scalar loads and each lane selects
      // its own; where the count is not a multiple of CL the last round's
      // spare lanes repeat the last partition and drop their result
      os << ind << "#pragma unroll 1\n" << ind << "for (int i2 = 0; i2 < " << (nit + CL - 1) / CL << "; ++i2) {\n";
      ind += "  ";
      for (int q = 0; q < CL; ++q)
        os << ind << "const int it" << q << " = " << CL << " * i2 + " << q << " < " << nit << " ? " << CL << " * i2 + " << q
           << " : " << nit - 1 << ";\n";
      for (int a = 0; a < P; ++a) {
        for (int q = 0; q < CL; ++q)
          os << ind << "int x" << q << "_" << a << " = " << ix_tab << "[it" << q << " * " << P << " + " << a
             << "]; asm volatile(\"\" : \"+s\"(x" << q << "_" << a << "));\n";
        std::string sel = "x" + std::to_string(CL - 1) + "_" + std::to_string(a);
        for (int q = CL - 2; q >= 0; --q)
          sel = "q_ == " + std::to_string(q) + " ? x" + std::to_string(q) + "_" + std::to_string(a) + " : (" + sel + ")";
        os << ind << "const int ix" << a << " = " << sel << ";\n";
        if (!k_lds) {
          const int nin = pr.i_eout - 1;
          os << ind << "const int sp" << a << " = ix" << a << " + (ix" << a << " < " << nin << " ? 1 : 2);\n";
          os << ind << "const double sg" << a << " = ix" << a << " < " << nin << " ? 1.0 : -1.0;\n";
          os << ind << "const double* const kp" << a << " = mom + (long long)(4 * sp" << a << ") * N + ptc;\n";
          for (int mu = 0; mu < 4; ++mu)
            os << ind << "const double k" << a << "_" << mu << " = kp" << a << "[" << mu << " * N];\n";
        }
      }
      if (nit % CL)
        for (auto& kv : acc_of_sum) {
          const int a = kv.second;
          os << ind << "const qx::cx<" << T << "> As" << a << " = A" << a << ";\n";
          if (v.prec != PREC_F64) os << ind << "const qx::cx<float> Cs" << a << " = C" << a << ";\n";
          if (abs_sum) os << ind << "const float Ss" << a << " = S" << a << ";\n";
        }
    }
    std::fill(done.begin(), done.end(), 0);
    kdone.clear();
    qdone.clear();
    qdone_d.clear();
    has_d.clear();
    double f0 = st.flops_per_point;
    bool was_local = (v.order & 4) != 0;
    (void)was_local;
    forward_block_inner(key, part[key]);
    // per lane: the loop's share of the partitions (the caller multiplies by
    // the lanes of a point)
    st.flops_per_point = f0 + pre + (st.flops_per_point - f0) * ((nit + CL - 1) / CL);
    if (cur_cache && nit % CL) {
      os << ind << "if (" << CL << " * i2 + q_ >= " << nit << ") {";
      for (auto& kv : acc_of_sum) {
        const int a = kv.second;
        os << " A" << a << " = As" << a << ";";
        if (v.prec != PREC_F64) os << " C" << a << " = Cs" << a << ";";
        if (abs_sum) os << " S" << a << " = Ss" << a << ";";
      }
      os << " }\n";
    }
    ind = outer;
    os << ind << "}\n";
    if (cur_cache && v.prec == PREC_F64) {
      // the point's lanes' partial amplitudes
      for (int o = 1; o < CL; o <<= 1)
        for (auto& kv : acc_of_sum)
          os << ind << "A" << kv.second << ".r += __shfl_xor(A" << kv.second << ".r, " << o << "); A" << kv.second
             << ".i += __shfl_xor(A" << kv.second << ".i, " << o << ");\n";
      st.flops_per_point += 2.0 * __builtin_ctz(CL) * (double)acc_of_sum.size();
    }
  }

  // Body: accumulators, all nodes in partition-grouped order, |A|^2 sums
  // added into the double `acc` of the enclosing scope.
  void body() {
    std::vector<int> sums = sum_nodes();
    for (size_t a = 0; a < sums.size(); ++a) {
      acc_of_sum[sums[a]] = (int)a;
      os << ind << "qx::cx<" << T << "> A" << a << " = {" << T << "(0), " << T << "(0)};\n";
      if (v.prec != PREC_F64) os << ind << "qx::cx<float> C" << a << " = {0.0f, 0.0f};\n";
      if (abs_sum) os << ind << "float S" << a << " = 0.0f;\n";
    }
    std::map<uint32_t, std::vector<int>> part;
    std::vector<uint32_t> order;
    partitions(part, order);
    if (mfma_join()) {
      mfma_body(part, order, (int)sums.size());
      return;
    }
    if (slot) {
      slot_loop(part);
    } else {
      if (r1_cache) emit_r1_cache();
      for (uint32_t key : order) forward_block(key, part[key]);
    }
    // |A|^2, summed over the enumerated configurations (HelSum) or single
    for (size_t a = 0; a < sums.size(); ++a) {
      if (v.prec == PREC_F64) {
        os << ind << "acc += A" << a << ".r * A" << a << ".r + A" << a << ".i * A" << a << ".i;\n";
      } else {
        os << ind << "{ double ar = (double)A" << a << ".r + (double)C" << a << ".r, ai = (double)A" << a
           << ".i + (double)C" << a << ".i;";
        if (abs_sum) os << " double sa = (double)S" << a << ";";
        if (cur_cache)
          // the point's lanes' partial sums, combined in FP64
          for (int o = 1; o < CL; o <<= 1) {
            os << " ar += __shfl_xor(ar, " << o << "); ai += __shfl_xor(ai, " << o << ");";
            if (abs_sum) os << " sa += __shfl_xor(sa, " << o << ");";
          }
        os << " acc += ar * ar + ai * ai;";
        if (abs_sum) os << " if (!(sa <= fix_kappa * fix_kappa * (ar * ar + ai * ai))) fixflag = 1;";
        os << " }\n";
      }
      st.flops_per_point += 4;
    }
  }

  // ---------------------------------------------------------------------
  // Join on the FP64 matrix cores (order flag 128; a measured experiment,
  // not a default).  Graphs whose every photon partition pairs 4 row
  // currents with 4 column currents, each pair the dot of a different one
  // of 16 amplitudes (the distributive helicity-sum graph with 4 photons
  // and the spins on lanes): per partition, each lane stores its row and
  // column currents in the wave's LDS staging area, and the 4 x 4 complex
  // dot matrices of two lanes at a time are computed by two
  // v_mfma_f64_4x4x4 (real part R_re J_re^T - R_im J_im^T and imaginary
  // part R_re J_im^T + R_im J_re^T, K = 4 spinor components).  Every
  // partition maps the 16 amplitudes to the 4 x 4 positions differently; a
  // lane permutation (__shfl) brings them to the first partition's layout
  // before they are accumulated.  The amplitudes are then gathered back to
  // their lanes through LDS for |A|^2.
  // ---------------------------------------------------------------------
  bool mfma_join() const { return (v.order & 128) != 0; }
  std::string mj_tab;  // kernel-name prefix of the per-partition permutation tables

  void mfma_body(std::map<uint32_t, std::vector<int>>& part, const std::vector<uint32_t>& order, int nsum) {
    if (v.prec != PREC_F64 || nsum != 16 || slot || stage())
      throw std::invalid_argument("the matrix-core join takes FP64 graphs with 16 amplitudes per lane");
    // per partition: row and column currents (index = position in the 4 x 4
    // block) and the amplitude of every position
    std::vector<std::array<int, 16>> pos_amp;
    std::vector<std::vector<int>> rows, cols;
    for (uint32_t key : order) {
      std::vector<int> B, J;
      std::array<int, 16> pa;
      pa.fill(-1);
      for (int k : part[key]) {
        const Node& dn = d.nodes[k];
        if (dn.kind != Kind::Dot) throw std::invalid_argument("matrix-core join: split joins only");
        auto ops = dot_ops(dn);
        int j = producer(ops.first), b = producer(ops.second);
        if (std::find(B.begin(), B.end(), b) == B.end()) B.push_back(b);
        if (std::find(J.begin(), J.end(), j) == J.end()) J.push_back(j);
        int r = (int)(std::find(B.begin(), B.end(), b) - B.begin());
        int c = (int)(std::find(J.begin(), J.end(), j) - J.begin());
        if (r > 3 || c > 3) throw std::invalid_argument("matrix-core join: a partition with more than 4 x 4 currents");
        int a = acc_of_sum.at(d.nodes[dn.out[0]].out[0]);
        if (pa[4 * r + c] >= 0) throw std::invalid_argument("matrix-core join: repeated dot");
        pa[4 * r + c] = a;
      }
      for (int x : pa)
        if (x < 0) throw std::invalid_argument("matrix-core join: incomplete 4 x 4 block");
      rows.push_back(B);
      cols.push_back(J);
      pos_amp.push_back(pa);
    }
    // position of every amplitude in the first partition (the accumulator layout)
    std::array<int, 16> pos0;
    for (int q = 0; q < 16; ++q) pos0[pos_amp[0][q]] = q;
    os << ind << "double mj[32];\n" << ind << "#pragma unroll\n" << ind << "for (int t = 0; t < 32; ++t) mj[t] = 0.0;\n";
    os << ind << "double* const mj_stg = qx_mj + (threadIdx.x >> 6) * " << 64 * kMjStride << ";\n";
    os << ind << "const int mj_lane = (int)(threadIdx.x & 63);\n";
    for (size_t p = 0; p < order.size(); ++p) {
      fence(1);
      os << ind << "// photons " << order[p] << " | " << (((1u << pr.P) - 1) & ~order[p])
         << " on the e-_in | e-_out side: 4 x 4 dots on the matrix cores\n";
      for (int b : rows[p]) emit(b);
      for (int j : cols[p]) emit(j);
      os << ind << "{\n";
      std::string o = ind;
      ind += "  ";
      os << ind << "double* const st_ = mj_stg + mj_lane * " << kMjStride << ";\n";
      for (int r = 0; r < 4; ++r)
        for (int k = 0; k < 4; ++k) {
          os << ind << "st_[" << 4 * r + k << "] = " << name(rows[p][r]) << ".c[" << k << "].r; st_[" << 16 + 4 * r + k
             << "] = " << name(rows[p][r]) << ".c[" << k << "].i;\n";
          os << ind << "st_[" << 32 + 4 * r + k << "] = " << name(cols[p][r]) << ".c[" << k << "].r; st_["
             << 48 + 4 * r + k << "] = " << name(cols[p][r]) << ".c[" << k << "].i;\n";
        }
      // source lane (within the lane's block) of the accumulator position
      // (i, j) = ((lane >> 4), lane & 3): where this partition put that amplitude
      os << ind << "const int src_ = " << mj_tab << "[" << p << " * 16 + ((mj_lane >> 4) << 2) + (mj_lane & 3)] + (mj_lane & 12);\n";
      os << ind << "qx::mfma_join4(mj_stg, " << kMjStride << ", src_, mj);\n";
      ind = o;
      os << ind << "}\n";
      st.flops_per_point += 16 * 32;
      st.n_dot += 16;
      (void)pos0;
    }
    // amplitudes back to their lanes, then |A|^2
    os << ind << "#pragma unroll\n" << ind << "for (int t = 0; t < 32; ++t) {\n";
    os << ind << "  const int blk_ = (mj_lane >> 2) & 3;\n";
    os << ind << "  mj_stg[(2 * t + (blk_ >> 1)) * " << kMjStride << " + (blk_ & 1) * 16 + (mj_lane >> 4) * 4 + (mj_lane & 3)] = mj[t];\n";
    os << ind << "}\n";
    os << ind << "#pragma unroll\n" << ind << "for (int q = 0; q < 32; ++q) { const double v_ = mj_stg[mj_lane * " << kMjStride
       << " + q]; acc += v_ * v_; }\n";
    st.flops_per_point += 16 * 4;
    // permutation tables: entry (i0, j0) of partition p is 16 i_p + j_p
    std::ostringstream tab;
    tab << "__constant__ int " << mj_tab << "[" << 16 * order.size() << "] = {";
    for (size_t p = 0; p < order.size(); ++p)
      for (int q0 = 0; q0 < 16; ++q0) {
        int a = pos_amp[0][q0];
        int qp = -1;
        for (int q = 0; q < 16; ++q)
          if (pos_amp[p][q] == a) qp = q;
        tab << (p || q0 ? ", " : "") << 16 * (qp >> 2) + (qp & 3);
      }
    tab << "};\n";
    mj_tables = tab.str();
  }
  std::string mj_tables;
  static constexpr int kMjStride = 65;  // doubles per lane in the staging area (padded against bank conflicts)

  // momenta for a partition-local block, opaque to the compiler
  void block_momenta() {
    if (batch_mom) {
      // loaded together: an empty asm takes 16 values at a time (short of
      // registers the compiler otherwise waits for each load in turn)
      os << ind << "long long pq = ptc;\n" << ind << "asm volatile(\"\" : \"+v\"(pq));\n";
      std::vector<std::string> ms;
      for (int p = 0; p < pr.npart; ++p)
        for (int mu = 0; mu < 4; ++mu) {
          ms.push_back("m" + std::to_string(p) + "_" + std::to_string(mu));
          os << ind << "double " << ms.back() << " = mom[" << (4 * p + mu) << " * N + pq];\n";
        }
      for (size_t i0 = 0; i0 < ms.size(); i0 += 16) {
        os << ind << "asm volatile(\"\" :";
        for (size_t i = i0; i < std::min(ms.size(), i0 + 16); ++i) os << (i > i0 ? ", " : " ") << "\"+v\"(" << ms[i] << ")";
        os << ");\n";
      }
    } else {
      os << ind << "long long pq = ptc;\n" << ind << "asm volatile(\"\" : \"+v\"(pq));\n";
      load_momenta("mom", "N", "pq");
    }
  }

  void load_momenta(const std::string& base, const std::string& N, const std::string& pt) {
    for (int p = 0; p < pr.npart; ++p)
      for (int mu = 0; mu < 4; ++mu)
        os << ind << "const double m" << p << "_" << mu << " = " << base << "[" << (4 * p + mu) << " * " << N
           << " + " << pt << "];\n";
  }

  // deposit the low bits of x into the positions of mask
  static std::string deposit(const std::string& x, uint32_t mask) {
    std::string s;
    int k = 0;
    for (int b = 0; b < 32; ++b)
      if ((mask >> b) & 1) {
        if (!s.empty()) s += " | ";
        s += "(((" + x + " >> " + std::to_string(k) + ") & 1u) << " + std::to_string(b) + ")";
        ++k;
      }
    return s.empty() ? "0u" : s;
  }

  // the per-lane part common to the kernel and the body function: helicity
  // code, loop over loop bits, graph body
  void lane_work(const std::string& hrt_expr) {
    os << ind << "const unsigned hrt = " << hrt_expr << ";\n";
    int nloop = popc(v.loop_mask);
    if (nloop > 0) {
      os << ind << "for (unsigned lp = 0; lp < " << (1u << nloop) << "u; ++lp) {\n";
      ind = "    ";
      os << ind << "const unsigned hc = hrt | " << deposit("lp", v.loop_mask) << ";\n";
      // order flag 32: momenta reloaded per iteration through an opaque index,
      // so nothing is hoisted out of the loop and kept live across it
      if (loop_local()) block_momenta();
      body();
      ind = "  ";
      os << ind << "}\n";
    } else {
      os << ind << "const unsigned hc = hrt;\n";
      body();
    }
  }
};

void check_variant(const Dag& d, const Variant& v) {
  uint32_t all = (1u << d.proc.npart) - 1;
  if (d.enum_mask != v.enum_mask) throw std::invalid_argument("graph/variant enumeration mismatch");
  if ((v.enum_mask & v.lane_mask) || (v.enum_mask & v.loop_mask) || (v.lane_mask & v.loop_mask))
    throw std::invalid_argument("helicity bit classes overlap");
  if (v.mode == HEL_SUM && (v.enum_mask | v.lane_mask | v.loop_mask) != all)
    throw std::invalid_argument("SUM mode must cover every helicity bit");
  if (v.mode == HEL_PER_POINT && (v.enum_mask | v.lane_mask | v.loop_mask) != 0)
    throw std::invalid_argument("PER_POINT mode takes every bit from the input");
  if (popc(v.lane_mask) > 6) throw std::invalid_argument("at most 64 lanes per point");
  if (v.order & 8)
    for (int a = 0; a < d.proc.P; ++a)
      if ((v.enum_mask >> d.proc.photon_particle[a]) & 1)
        throw std::invalid_argument("the partition loop takes photon helicities at run time only");
  if (v.block % 64 != 0 || v.block < 64 || v.block > 1024) throw std::invalid_argument("bad block size");
  if (((v.order & (256 | 512)) &&
       ((v.order & 256 && v.order & 512) || !(v.order & 8) || v.mode != HEL_PER_POINT || (v.order & 64) ||
        v.lane_mask || d.split < 2 || d.proc.P - d.split < 1 || d.distributed)) ||
      ((v.order & 1024) && !(v.order & (256 | 512))) || ((v.order & 8192) && !(v.order & 4)) ||
      ((v.order & 2048) && (v.mode != HEL_SUM || v.lane_mask != (1u << d.proc.i_eout) ||
                            !((v.enum_mask >> d.proc.i_ein) & 1u) || (v.order & (8 | 16 | 128)) || d.distributed)))
    throw std::invalid_argument(
        "the one-photon current cache takes per-point partition loops with split >= 2; the shared e-_in side "
        "takes helicity sums with the e-_out spin as the one lane bit and the e-_in spin in the graph; batched "
        "block momenta take per-partition blocks");
}

// The one-photon current cache of a variant for BP points per LDS region
// whose budget is `budget` bytes: sets e's cache fields; throws if even the
// currents and polarisations do not fit.
void setup_cache(Emitter& e, const Dag& d, const Variant& v, const std::string& kname, int BP, int64_t budget) {
  e.cur_cache = true;
  e.CL = cache_lanes(v);
  e.BP = BP;
  e.ix_tab = kname + "_ix";
  e.row_only = (v.order & 1024) != 0;
  const int64_t per = (int64_t)d.proc.P * BP;                  // photon-points
  const int tsz = v.prec == PREC_F64 ? 8 : 4;                   // currents, polarisations
  const int ncur = e.row_only ? 8 : 16;
  if ((ncur + 3) * tsz * per > budget) throw std::invalid_argument("the current cache does not fit the LDS");
  e.k_lds = ((ncur + 3) * tsz + 4 * 8) * per <= budget;        // momenta in FP64
}

// Bytes of the cache's three arrays for BP points (polarisations and
// currents in the graph's type, momenta in FP64).
int64_t cache_bytes(const Emitter& e, const Dag& d, const Variant& v) {
  const int tsz = v.prec == PREC_F64 ? 8 : 4;
  return (((e.row_only ? 8 : 16) + 3) * tsz + (e.k_lds ? 32 : 0)) * (int64_t)d.proc.P * e.BP;
}

}  // namespace

int body_cache_doubles(const Dag& d, const Variant& v) {
  if (!(v.order & (256 | 512))) return 0;
  Emitter e(d, v);
  setup_cache(e, d, v, "", 64 / cache_lanes(v), kBodyCacheBytes);
  return (int)((cache_bytes(e, d, v) + 7) / 8);
}

std::string emit_eval_kernel(const Dag& d, const Variant& v, const std::string& kname, EmitStats* stats) {
  check_variant(d, v);
  Emitter e(d, v);
  const int G = lanes_per_point(v);
  const int LB = __builtin_ctz(G);
  std::ostringstream& os = e.os;
  os << "// generated by qedx: " << variant_tag(v, d.proc.n_out, d.proc.n_in) << "\n";
  os << "#include <hip/hip_runtime.h>\n";
  os << device_header_text() << "\n";
  if (v.fixup) {
    if (v.prec != PREC_F32C || v.mode != HEL_PER_POINT)
      throw std::invalid_argument("the FP64 fix-up is built for FP32C per-point kernels");
    if (v.order & 16) throw std::invalid_argument("the FP64 fix-up excludes LDS staging");
    e.abs_sum = true;
  }
  if (v.order & 8) {
    e.slot = true;
    e.pol_lds = true;
    e.slot_tab = kname + "_slots";
    if (v.order & (256 | 512)) {
      // polarisations (3), currents (16, or 8 for the e-_in side only) and
      // momenta (4) per photon and point; the momenta only where the
      // workgroups that min_waves asks for still fit the 160 KB of LDS of a
      // compute unit (4 SIMDs)
      const int64_t budget = (int64_t)160 * 1024 * v.block / (256 * std::max(1, v.min_waves));
      setup_cache(e, d, v, kname, v.block / cache_lanes(v), budget);
    }
    e.emit_slot_table();
  }
  if (v.order & 2048) {
    e.coop = true;
    e.build_twins();
  }
  e.batch_mom = (v.order & 8192) != 0;
  if (v.order & 4096) {
    if (!(v.order & 2048) || !(v.order & 4) || v.prec != PREC_F64)
      throw std::invalid_argument("the e-_in-side current cache takes FP64 helicity sums with the shared e-_in side");
    e.r1_cache = true;
    e.r1_collect();
  }
  e.mj_tab = kname + "_mjperm";
  const std::string mj_mark = "//@MJTAB@\n";
  if (e.mfma_join()) {
    if (v.block != 256) throw std::invalid_argument("the matrix-core join takes 256-lane workgroups");
    os << mj_mark;
  }
  os << "extern \"C\" __global__ void __launch_bounds__(" << v.block;
  if (v.min_waves > 0) os << ", " << v.min_waves;
  os << ")\n" << kname
     << "(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, double* __restrict__ out"
     << (v.fixup ? ", double fix_kappa" : "") << ")\n{\n";
  const std::string lds_mark = "  //@LDS@\n";
  os << lds_mark;
  os << "  const long long gid = (long long)blockIdx.x * " << v.block << " + threadIdx.x;\n";
  os << "  const long long pt = gid >> " << LB << ";\n";
  os << "  const unsigned sub = (unsigned)(gid & " << (G - 1) << ");\n";
  os << "  const long long ptc = pt < N ? pt : N - 1;\n";
  if (!e.local() && !e.slot && !e.loop_local()) e.load_momenta("mom", "N", "ptc");
  os << "  double acc = 0.0;\n";
  if (v.fixup) os << "  int fixflag = 0;\n";
  std::string hrt = v.mode == HEL_PER_POINT ? "hel[ptc]" : Emitter::deposit("sub", v.lane_mask);
  e.lane_work(hrt);
  // helicity lanes hold parts of the sum (the cache's two lanes hold the
  // same |A|^2, their amplitudes already combined)
  for (int o = e.CL; o < G; o <<= 1) os << "  acc += __shfl_xor(acc, " << o << ");\n";
  if (v.fixup)
    // a point the FP32 pass cannot resolve is marked in place with a negative
    // value (|M|^2 itself is never negative); the FP64 pass below finds it
    os << "  if (pt < N && sub == 0u) out[pt] = fixflag ? -1.0 : acc;\n}\n";
  else
    os << "  if (pt < N && sub == 0u) out[pt] = acc;\n}\n";
  // per point: every lane of the group does the body once per loop iteration
  e.st.flops_per_point *= (double)G * (double)(1 << popc(v.loop_mask));
  std::string src = os.str();
  {
    // per-lane LDS slots for staged currents: [slot][8 words][block]
    std::string decl;
    if (e.lds_slots > 0)
      decl = "  __shared__ " + e.T + " qx_lds[" + std::to_string(e.lds_slots * 8 * v.block) + "];\n";
    if (e.cur_cache) {
      decl += "  __shared__ " + e.T + " qx_pol[" + std::to_string(3 * d.proc.P * e.BP) + "];\n";
      decl += "  __shared__ " + e.T + " qx_cur[" + std::to_string((e.row_only ? 8 : 16) * d.proc.P * e.BP) + "];\n";
      if (e.k_lds) decl += "  __shared__ double qx_k[" + std::to_string(4 * d.proc.P * e.BP) + "];\n";
    } else if (e.pol_lds) {
      decl += "  __shared__ " + e.PT + " qx_pol[" + std::to_string(3 * d.proc.npart * v.block) + "];\n";
    }
    if (e.mfma_join()) decl += "  __shared__ double qx_mj[" + std::to_string(4 * 64 * Emitter::kMjStride) + "];\n";
    if (e.r1_cache) decl += "  __shared__ double qx_r1[" + std::to_string(8 * e.r1_slot.size() * v.block) + "];\n";
    size_t at = src.find(lds_mark);
    src.replace(at, lds_mark.size(), decl);
    if (e.mfma_join()) src.replace(src.find(mj_mark), mj_mark.size(), e.mj_tables);
  }
  if (v.fixup) {
    // FP64 pass over the points the FP32C kernel could not resolve
    Variant v64 = v;
    v64.prec = PREC_F64;
    v64.fixup = 0;
    v64.min_waves = 0;
    EmitStats st64;
    std::ostringstream fx;
    const bool pair = pair_kernel(d.proc, v64);
    if (pair)
      fx << subset_header_text() << "\n" << emit_pair_body(d.proc, kname + "_b64", &st64) << "\n";
    else
      fx << emit_body_function(d, v64, kname + "_b64", &st64) << "\n";
    // the pair body, and the FP64 body with the one-photon current cache,
    // take CL lanes per point and their wave's LDS region
    const int CL = pair ? 2 : cache_lanes(v64);
    const int W = pair ? pair_lds_doubles(d.proc) : body_cache_doubles(d, v64);
    // Each workgroup of 256 lanes owns kFixRange consecutive points: it scans
    // their results for the negative marks, compacts the marked offsets in
    // LDS (one LDS atomic per wave: ballot, then each marked lane's rank
    // among the marked lanes below it) and recomputes them 256 / CL at a
    // time, so the FP64 body runs on full waves however sparse the marks are.
    fx << "extern \"C\" __global__ void __launch_bounds__(256)\n"
       << kname << "_fix(const double* __restrict__ mom, const unsigned* __restrict__ hel, long long N, "
       << "double* __restrict__ out)\n{\n"
       << (W ? "  __shared__ double2 qx_fc[" + std::to_string(2 * W) + "];\n" : std::string())
       << "  __shared__ unsigned short fx_list[" << kFixRange << "];\n"
       << "  __shared__ unsigned fx_cnt;\n"
       << "  if (threadIdx.x == 0) fx_cnt = 0u;\n"
       << "  __syncthreads();\n"
       << "  const long long base = (long long)blockIdx.x * " << kFixRange << ";\n"
       << "  const unsigned ln_ = __lane_id();\n"
       << "  for (unsigned i = threadIdx.x; i < " << kFixRange << "u; i += 256u) {\n"
       << "    const long long pt = base + (long long)i;\n"
       << "    const bool f_ = pt < N && out[pt] < 0.0;\n"
       << "    const unsigned long long fm_ = __ballot(f_);\n"
       << "    if (fm_) {\n"
       << "      const unsigned ld_ = (unsigned)__ffsll((unsigned long long)fm_) - 1u;\n"
       << "      unsigned b_ = 0u;\n"
       << "      if (ln_ == ld_) b_ = atomicAdd(&fx_cnt, (unsigned)__popcll(fm_));\n"
       << "      b_ = __shfl(b_, (int)ld_);\n"
       << "      if (f_) fx_list[b_ + (unsigned)__popcll(fm_ & ((1ull << ln_) - 1ull))] = (unsigned short)i;\n"
       << "    }\n"
       << "  }\n"
       << "  __syncthreads();\n"
       << "  const unsigned cnt = fx_cnt;\n";
    if (CL == 1) {
      fx << "  for (unsigned j = threadIdx.x; j < cnt; j += 256u) {\n"
         << "    const long long pt = base + (long long)fx_list[j];\n"
         << "    out[pt] = " << kname << "_b64(mom, N, pt, hel[pt]);\n"
         << "  }\n}\n";
    } else {
      // every lane takes part in every round (the body synchronises its wave)
      const int sh = __builtin_ctz(CL);
      fx << "  const unsigned sub = threadIdx.x & " << CL - 1 << "u;\n"
         << "  for (unsigned j0 = 0; j0 < cnt; j0 += " << 256 / CL << "u) {\n"
         << "    const unsigned j = j0 + (threadIdx.x >> " << sh << ");\n"
         << "    const long long pt = base + (long long)fx_list[j < cnt ? j : cnt - 1u];\n"
         << "    const double r = " << kname << "_b64(mom, "
         << (pair ? "hel, N, pt, " : "N, pt, hel[pt], ")
         << (W ? "(double*)qx_fc + (threadIdx.x >> 6) * " + std::to_string(W) : std::string("nullptr"))
         << (pair ? std::string() : ", (int)((threadIdx.x & 63u) >> " + std::to_string(sh) + "), sub") << ");\n"
         << "    if (j < cnt && sub == 0u) out[pt] = r;\n"
         << "  }\n}\n";
    }
    src += fx.str();
  }
  e.st.lines = std::count(src.begin(), src.end(), '\n');
  if (stats) *stats = e.st;
  return src;
}

std::string emit_body_function(const Dag& d, const Variant& v, const std::string& fname, EmitStats* stats,
                               bool pol_param) {
  check_variant(d, v);
  if (v.order & 16) throw std::invalid_argument("LDS staging is built for eval kernels only");
  Emitter e(d, v);
  std::ostringstream& os = e.os;
  if (v.order & 8) {
    e.slot = true;
    e.pol_lds = pol_param;
    e.slot_tab = fname + "_slots";
    if (v.order & (256 | 512)) {
      setup_cache(e, d, v, fname, 64 / cache_lanes(v), kBodyCacheBytes);
      e.body_mode = true;
      e.pol_lds = true;
    }
    e.emit_slot_table();
  }
  if (v.fixup) {
    if (v.prec != PREC_F32C || v.mode != HEL_PER_POINT)
      throw std::invalid_argument("the FP64 fix-up is built for FP32C per-point bodies");
    e.abs_sum = true;
  }
  os << "static __device__ double " << fname
     << "(const double* __restrict__ mom, long long N, long long ptc, unsigned hrt_in"
     << (e.cur_cache ? ", double* __restrict__ qx_c, int tpt, unsigned sub"
                     : e.pol_lds ? ", " + e.PT + "* __restrict__ qx_pol" : std::string())
     << (v.fixup ? ", int& fixflag, double fix_kappa" : "") << ")\n{\n";
  if (e.cur_cache) {
    const int P = d.proc.P, ncur = e.row_only ? 8 : 16;
    // (3 + ncur) P BP is even (BP is a multiple of 16), so qx_k stays 8-byte aligned
    os << "  " << e.T << "* const qx_pol = (" << e.T << "*)qx_c;\n";
    os << "  " << e.T << "* const qx_cur = qx_pol + " << 3 * P * e.BP << ";\n";
    if (e.k_lds) os << "  double* const qx_k = (double*)(qx_cur + " << ncur * P * e.BP << ");\n";
  }
  if (!e.local() && !e.slot) e.load_momenta("mom", "N", "ptc");
  os << "  double acc = 0.0;\n";
  e.lane_work("hrt_in");
  os << "  return acc;\n}\n";
  e.st.flops_per_point *= (double)lanes_per_point(v) * (double)(1 << popc(v.loop_mask));
  if (stats) *stats = e.st;
  return os.str();
}

}  // namespace qedx
