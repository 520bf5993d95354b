// qedx_batch.cpp -- mixed-process batches: one persistent kernel over
// segments of different processes, replayed from a captured HIP graph.
//
// Work is cut into tiles of 64 * chunk lanes of one segment, laid out by
// decreasing cost per point (the static FLOP count of the kernels).  Each
// wavefront takes its share of the tile space, cut on the host to equal cost -- a
// contiguous range of tiles (pair kernels), or some rounds of each segment (other
// modules) -- and evaluates it with the bodies of its segments' processes.  Grid size and tile length are
// picked by timing a few candidates once per plan signature; the choice is
// kept in autotune.txt in the code-object cache directory.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "qedx_internal.hpp"
#include "qedx_pair.hpp"

using namespace qedx;
using qedx_rt::fail;

namespace {

struct DevSeg {  // mirrored by qedx_seg in the generated module
  const double* mom;
  const uint32_t* hel;
  double* out;
  long long N;
  long long tile0;
  int proc;
  int shift;       // log2 of the process body's lanes per point
  int shift64;     // ... of its body in the FP32C fix-up pass
  long long list0; // FP32C fix-up: the segment's region of the point list
};

// A process's variant as a body of the persistent kernel: the eval kernel's
// shape without its occupancy hint (the batch kernel has its own launch
// bounds).
Variant batch_variant(Variant v) {
  v.min_waves = 0;
  return v;
}

// FP32C per-point modules with the FP64 fix-up (every process of a batch
// shares the precision, so the first one decides): the batch kernel lists
// the points whose diagram sum cancels, per segment (a counter per segment,
// the segment's region of the list), and qedx_batch_fix recomputes them in FP64
// (pair bodies, or of the same graphs where a kernel shape is given), one
// segment at a time per wave, so bodies that split a point over several lanes
// run there too.
bool module_fixup(const std::vector<std::pair<Process, Variant>>& procs) {
  return !procs.empty() && procs[0].second.fixup != 0;
}

std::string module_source(const std::vector<std::pair<Process, Variant>>& procs) {
  const bool fix = module_fixup(procs);
  std::ostringstream os;
  os << "// generated by qedx: mixed-process batch module\n#include <hip/hip_runtime.h>\n";
  os << device_header_text() << "\n";
  // the 7-photon body keeps its photon polarisations in one per-lane LDS
  // array of the batch kernel (3 npart values per lane), as the eval kernels
  // do; for every slot-loop body it raised the batch kernel's registers into
  // scratch (5.9 against 5.5 ms on the FP64 n = 1..6 batch), for the n = 6
  // body alone it has no scratch and is 4.5 % faster (5.34 against 5.58 ms).
  // A 7-photon pair body in the same kernel takes 156 of a workgroup's 160 KB:
  // the polarisations stay in registers there.
  // Bodies with the one-photon current cache (FP64 per point, 5..7 photons)
  // run 2 or 4 lanes per point and keep the cache in their wave's region of
  // qx_cache_mem.
  // FP64 processes without an explicit kernel shape take the pair bodies (two
  // lanes per point; pair), and so does the FP64 pass of such FP32C processes
  // (pair64).
  std::vector<char> pol(procs.size(), 0), cache(procs.size(), 0), cache64(procs.size(), 0), pair(procs.size(), 0),
      pair64(procs.size(), 0);
  os << subset_header_text() << "\n";
  int pol_npart = 0, cache_w = 0, cache_w64 = 0;
  bool pol_fits = true;
  for (auto& p : procs) pol_fits = pol_fits && !(pair_eval(p.first, p.second) && pair_lds_doubles(p.first) > 0);
  for (size_t i = 0; i < procs.size(); ++i) {
    Dag d = graph_for(procs[i].first, procs[i].second, nullptr, nullptr);
    EmitStats st;
    const Process& pr = procs[i].first;
    pair[i] = pair_eval(pr, procs[i].second);
    pair64[i] = fix && pair_kernel(pr, procs[i].second);
    if (pair[i]) {
      cache_w = std::max(cache_w, pair_lds_doubles(pr));
      os << emit_pair_body(pr, "qedx_body_" + std::to_string(i), &st) << "\n";
      continue;
    }
    const int cw = body_cache_doubles(d, procs[i].second);
    cache[i] = cw > 0;
    cache_w = std::max(cache_w, cw);
    pol[i] = pol_fits && !cache[i] && (procs[i].second.order & 8) && procs[i].second.block == 256 && procs[i].first.P >= 7;
    if (pol[i]) pol_npart = std::max(pol_npart, procs[i].first.npart);
    os << emit_body_function(d, procs[i].second, "qedx_body_" + std::to_string(i), &st, pol[i] != 0) << "\n";
    if (fix) {
      Variant v64 = procs[i].second;
      v64.prec = PREC_F64;
      v64.fixup = 0;
      if (pair64[i]) {
        cache_w64 = std::max(cache_w64, pair_lds_doubles(pr));
        os << emit_pair_body(pr, "qedx_body64_" + std::to_string(i), &st) << "\n";
        continue;
      }
      const int cw64 = body_cache_doubles(d, v64);
      cache64[i] = cw64 > 0;
      cache_w64 = std::max(cache_w64, cw64);
      os << emit_body_function(d, v64, "qedx_body64_" + std::to_string(i), &st) << "\n";
    }
  }
  os << "struct qedx_seg { const double* mom; const unsigned* hel; double* out; long long N; long long tile0; "
        "int proc; int shift; int shift64; long long list0; };\n";
  os << "extern \"C\" __global__ void __launch_bounds__(256)\n"
        "qedx_batch(const qedx_seg* __restrict__ segs, const int* __restrict__ share"
     << (fix ? ", double fix_kappa, unsigned* __restrict__ fix_cnt, unsigned* __restrict__ fix_list" : "")
     << ")\n{\n";
  std::string PT = "double";
  for (size_t i = 0; i < procs.size(); ++i)
    if (pol[i]) PT = pol_lds_type(procs[i].second);
  if (pol_npart > 0) os << "  __shared__ " << PT << " qx_pol_mem[" << 3 * pol_npart * 256 << "];\n";
  if (cache_w > 0) os << "  __shared__ double2 qx_cache_mem[" << 2 * cache_w << "];\n";
  os << "  const int lane = threadIdx.x & 63;\n";
  os << "  const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4u + (threadIdx.x >> 6)));\n";
  // the wave's share: entries (segment, first round of 64 lanes, rounds) in [share[w], share[w + 1])
  os << "  const int last = share[w + 1];\n  for (int e = share[w]; e < last; e += 3) {\n";
  os << "    const int s = share[e];\n    const qedx_seg sg = segs[s];\n";
  os << "    const int lp = lane >> sg.shift;\n";
  os << "    const unsigned sub = (unsigned)(lane & ((1 << sg.shift) - 1));\n";
  os << "    const long long ppw = 64LL >> sg.shift, end = (long long)share[e + 1] + share[e + 2];\n";
  os << "    for (long long t = share[e + 1]; t < end; ++t) {\n";
  os << "      const long long pt = t * ppw + lp;\n";
  os << "      const long long ptc = pt < sg.N ? pt : sg.N - 1;\n";
  os << "      const unsigned hrt = sg.hel[ptc];\n";
  os << "      double r = 0.0;\n";
  if (fix) os << "      int ff = 0;\n";
  os << "      switch (sg.proc) {\n";
  for (size_t i = 0; i < procs.size(); ++i)
    if (pair[i])
      os << "        case " << i << ": r = qedx_body_" << i << "(sg.mom, sg.hel, sg.N, ptc, "
         << (cache_w ? "(double*)qx_cache_mem + (threadIdx.x >> 6) * " + std::to_string(cache_w) : "nullptr") << "); break;\n";
    else
      os << "        case " << i << ": r = qedx_body_" << i << "(sg.mom, sg.N, ptc, hrt"
         << (cache[i] ? ", (double*)qx_cache_mem + (threadIdx.x >> 6) * " + std::to_string(cache_w) + ", lp, sub"
                      : pol[i] ? ", qx_pol_mem" : "")
         << (fix ? ", ff, fix_kappa" : "") << "); break;\n";
  os << "        default: break;\n      }\n";
  os << "      if (pt < sg.N && sub == 0u) sg.out[pt] = r;\n";
  if (fix) {
    // one counter update per wave; entries are the segment's point indices
    os << "      const bool fx_ = ff && pt < sg.N && sub == 0u;\n"
       << "      const unsigned long long fm_ = __ballot(fx_);\n"
       << "      if (fm_) {\n"
       << "        const unsigned ld_ = (unsigned)__ffsll((unsigned long long)fm_) - 1u;\n"
       << "        unsigned base_ = 0u;\n"
       << "        if ((unsigned)lane == ld_) base_ = atomicAdd(fix_cnt + s, (unsigned)__popcll(fm_));\n"
       << "        base_ = __shfl(base_, (int)ld_);\n"
       << "        if (fx_) {\n"
       << "          const size_t k_ = (size_t)base_ + (size_t)__popcll(fm_ & ((1ull << lane) - 1ull));\n"
       << "          fix_list[sg.list0 + (long long)k_] = (unsigned)pt;\n"
       << "        }\n      }\n";
  }
  os << "    }\n  }\n}\n";
  // clears the 64 counters at c (fix-up points of the segments)
  if (fix)
    os << "extern \"C\" __global__ void qedx_zero(unsigned* __restrict__ c)\n{\n"
          "  if (blockIdx.x == 0 && threadIdx.x < 64) c[threadIdx.x] = 0u;\n}\n";
  if (fix) {
    // every wave walks the segments in turn and takes its share of each
    // segment's list, 64 >> shift points per round (all lanes take part in
    // every round: a body that splits a point synchronises its wave)
    os << "extern \"C\" __global__ void __launch_bounds__(256)\n"
          "qedx_batch_fix(const qedx_seg* __restrict__ segs, int nseg, const unsigned* __restrict__ fix_cnt, "
          "const unsigned* __restrict__ fix_list)\n{\n";
    if (cache_w64 > 0) os << "  __shared__ double2 qx_fc[" << 2 * cache_w64 << "];\n";
    os << "  const int lane = threadIdx.x & 63;\n"
          "  const long long wave = (long long)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (long long)gridDim.x * 4;\n"
          "  for (int s = 0; s < nseg; ++s) {\n"
          "    const qedx_seg sg = segs[s];\n"
          "    const long long cnt = (long long)fix_cnt[s];\n"
          "    const int lp = lane >> sg.shift64;\n"
          "    const unsigned sub = (unsigned)(lane & ((1 << sg.shift64) - 1));\n"
          "    const long long ppw = 64LL >> sg.shift64;\n"
          "    for (long long j0 = wave * ppw; j0 < cnt; j0 += nwaves * ppw) {\n"
          "      const long long j = j0 + lp;\n"
          "      const long long pt = (long long)fix_list[sg.list0 + (j < cnt ? j : cnt - 1)];\n"
          "      double r = 0.0;\n"
          "      switch (sg.proc) {\n";
    for (size_t i = 0; i < procs.size(); ++i)
      if (pair64[i])
        os << "        case " << i << ": r = qedx_body64_" << i << "(sg.mom, sg.hel, sg.N, pt, "
           << (cache_w64 ? "(double*)qx_fc + (threadIdx.x >> 6) * " + std::to_string(cache_w64) : "nullptr") << "); break;\n";
      else
        os << "        case " << i << ": r = qedx_body64_" << i << "(sg.mom, sg.N, pt, sg.hel[pt]"
           << (cache64[i] ? ", (double*)qx_fc + (threadIdx.x >> 6) * " + std::to_string(cache_w64) + ", lp, sub" : "")
           << "); break;\n";
    os << "        default: break;\n      }\n"
          "      if (j < cnt && sub == 0u) sg.out[pt] = r;\n    }\n  }\n}\n";
  }
  return os.str();
}

// ---------------------------------------------------------------------------
// Plans whose processes all take the pair kernels (FP64, no kernel shape asked
// for) share one module for n = 1..6, so no plan waits for a compiler (an empty
// code-object cache does, 19 s, where a module of n = 1 alone took 1).  It
// holds a kernel for all processes, for batches too small to fill the device,
// and one per class of processes with registers and LDS of that class: in the
// common kernel the 7-photon body leaves every other one a single wave per
// SIMD and none of the LDS.  A wave's tiles are a contiguous range of the tile
// space, cut on the host by the segments' cost: taking them from a counter
// cost 5.8 ns per tile in the counter's memory alone (86,000 tiles of the
// n = 1..6 batch: 1.43 ms, and 0.94 ms with four rounds of points per tile),
// and a range's next inputs can be loaded ahead.
// ---------------------------------------------------------------------------
struct PairClass {
  const char* name;
  int lo, hi;  // outgoing photons
  int waves;   // waves per SIMD
};
const PairClass kPairClasses[] = {{"qedx_batch_n6", 6, 6, 1}, {"qedx_batch_n45", 4, 5, 1}, {"qedx_batch_n13", 1, 3, 2}};
const int kClasses = 3;
int pair_class(int n) { return n == 6 ? 0 : n >= 4 ? 1 : 2; }

std::string pair_module_source() {
  std::ostringstream os;
  os << "// generated by qedx: mixed-process batch module\n" << kContractOn << "#include <hip/hip_runtime.h>\n";
  os << device_header_text() << "\n" << subset_header_text() << "\n";
  os << "struct qedx_seg { const double* mom; const unsigned* hel; double* out; long long N; long long tile0; "
        "int proc; int shift; int shift64; long long list0; };\n";
  for (int n = 1; n <= 6; ++n) {
    const Process pr = Process::make(n, 1);
    const std::string b = "qedx_body_" + std::to_string(n);
    EmitStats st;
    os << emit_pair_body(pr, b, &st) << "\n";
    // `rounds` times 32 points; up to 6 photons the next round's inputs are
    // loaded while this one's are worked on
    os << "static __device__ __forceinline__ void qedx_run_" << n
       << "(const qedx_seg& sg, long long p0, long long rounds, double* __restrict__ lds)\n{\n";
    if (pair_persistent(pr)) {
      os << "  const long long end = p0 + 32 * rounds;\n  " << b
         << "_tiles(sg.mom, sg.hel, sg.N, sg.out, p0, 32, end < sg.N ? end : sg.N, lds);\n}\n";
      continue;
    }
    os << "  long long pt = p0 + (__lane_id() >> 1);\n";
    os << "  " << b << "_in cur;\n  " << b << "_load(sg.mom, sg.hel, sg.N, pt < sg.N ? pt : sg.N - 1, cur);\n";
    os << "  while (true) {\n    const bool more = --rounds > 0;\n    const long long nx = pt + 32;\n";
    if (n < 6) {
      os << "    " << b << "_in nin = cur;\n    if (more) " << b << "_load(sg.mom, sg.hel, sg.N, nx < sg.N ? nx : sg.N - 1, nin);\n";
      os << "    __builtin_amdgcn_sched_barrier(0);\n";
    }
    os << "    const double r = " << b << "_run(cur, lds);\n";
    os << "    if (pt < sg.N && (__lane_id() & 1u) == 0u) sg.out[pt] = r;\n";
    os << "    if (!more) break;\n    pt = nx;\n";
    if (n < 6)
      os << "    cur = nin;\n";
    else
      os << "    " << b << "_load(sg.mom, sg.hel, sg.N, pt < sg.N ? pt : sg.N - 1, cur);\n";
    os << "  }\n}\n";
  }
  auto kernel = [&](const std::string& name, int lo, int hi, int waves) {
    int W = 0;
    for (int n = lo; n <= hi; ++n) W = std::max({W, pair_lds_doubles(Process::make(n, 1)), pair_in_doubles(Process::make(n, 1))});
    os << "extern \"C\" __global__ void __launch_bounds__(256, " << waves << ")\n" << name
       << "(const qedx_seg* __restrict__ segs, int nseg, const long long* __restrict__ cut, int chunk)\n{\n";
    if (W) os << "  __shared__ double2 qx_lds[" << 2 * W << "];\n";
    os << "  double* const lds = " << (W ? "(double*)qx_lds + (threadIdx.x >> 6) * " + std::to_string(W) : std::string("nullptr"))
       << ";\n";
    os << "  const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4u + (threadIdx.x >> 6)));\n";
    os << "  long long t = cut[w];\n  const long long end = cut[w + 1];\n  int s = 0;\n  while (t < end) {\n";
    os << "    while (s + 1 < nseg && segs[s + 1].tile0 <= t) ++s;\n";
    os << "    const qedx_seg sg = segs[s];\n";
    os << "    const long long stop = s + 1 < nseg && segs[s + 1].tile0 < end ? segs[s + 1].tile0 : end;\n";
    os << "    const long long p0 = (t - sg.tile0) * 32 * chunk, left = (sg.N - p0 + 31) >> 5, all = (stop - t) * chunk;\n";
    os << "    const long long rounds = all < left ? all : left;\n    t = stop;\n    switch (sg.proc) {\n";
    for (int n = lo; n <= hi; ++n) os << "      case " << n << ": qedx_run_" << n << "(sg, p0, rounds, lds); break;\n";
    os << "      default: break;\n    }\n  }\n}\n";
  };
  kernel("qedx_batch", 1, 6, 1);
  for (const PairClass& c : kPairClasses) kernel(c.name, c.lo, c.hi, c.waves);
  return os.str();
}

// Relative time of a point: its FLOPs, and 1500 more for what the smallest
// processes wait for.
double tile_cost(double flops_per_point) { return flops_per_point + 1500.0; }

// A lane's time with a point's share in the other modules' kernels: its FLOPs,
// and 3500 more.  (FP32C, us per round of n = 1..6: 8.2, 11.6, 19, 35, 60, 271;
// FLOPs per lane 484, 1332, 3972, 10492, 19932, 112748.)
constexpr double kLaneCost = 3500.0;

bool all_pair(const std::vector<std::pair<Process, Variant>>& pv) {
  for (auto& p : pv)
    if (p.first.n_in != 1 || !pair_eval(p.first, p.second)) return false;
  return true;
}

std::string batch_tag(const std::vector<std::pair<Process, Variant>>& pv) {
  if (all_pair(pv)) return "batch_pair_f64";
  std::string tag = "batch";
  for (auto& p : pv) tag += "_n" + std::to_string(p.first.n_out) + (p.second.rewrite ? "d" + std::to_string(p.second.rewrite) : "");
  tag += pv.empty() || pv[0].second.prec == PREC_F64 ? "_f64" : "_f32c";
  if (module_fixup(pv)) tag += "_fx";
  return tag;
}

std::mutex g_tune_mu;

std::string tune_path() { return qedx_rt::cache_dir() + "/autotune.txt"; }

bool tune_lookup(const std::string& key, int& grid, int& chunk) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  std::ifstream f(tune_path());
  std::string k;
  int g, c;
  while (f >> k >> g >> c)
    if (k == key) {
      grid = g;
      chunk = c;
      return true;
    }
  return false;
}

void tune_store(const std::string& key, int grid, int chunk) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  std::ofstream f(tune_path(), std::ios::app);
  f << key << " " << grid << " " << chunk << "\n";
}

}  // namespace

struct qed_batch_plan {
  bool pair = false;      // the module of the pair kernels
  bool classes = false;   // ... one kernel per class of processes
  hipFunction_t f_class[kClasses] = {};
  long long cls_tile[kClasses + 1] = {};  // tiles of a class
  int* d_share = nullptr;                 // other modules: the waves' shares (see their kernel)
  long long* d_cut = nullptr;             // first tile of every wave, and the end, of each kernel in turn
  int cut_at[kClasses] = {}, cut_groups[kClasses] = {};  // ... where a kernel's start, its workgroups
  int ncu = 256;
  hipModule_t mod = nullptr;
  hipFunction_t f_batch = nullptr, f_zero = nullptr, f_fix = nullptr;
  DevSeg* d_segs = nullptr;
  unsigned* d_fix = nullptr;  // FP32C fix-up: [64 per-segment counts, point lists of the segments]
  double fix_kappa = 0;
  long long fix_grid = 0;
  int nseg = 0;
  long long ntiles = 0;
  int chunk = 1;
  int grid = 0;  // workgroups of 256 threads (pair module: autotune's choice, 0 = a kernel per class)
  std::vector<int> shift, shift64;  // per distinct process: log2 of its bodies' lanes per point
  hipStream_t cap = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  std::vector<DevSeg> host;
  ~qed_batch_plan() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (cap) {
      (void)hipStreamSynchronize(cap);
      (void)hipStreamDestroy(cap);
    }
    if (d_segs) (void)hipFree(d_segs);
    if (d_cut) (void)hipFree(d_cut);
    if (d_share) (void)hipFree(d_share);
    if (d_fix) (void)hipFree(d_fix);
    if (mod) (void)hipModuleUnload(mod);
  }
};

static qed_status launch_eager(qed_batch_plan* b, hipStream_t s) {
  hipError_t e;
  if (b->pair) {
    for (int c = 0; c < (b->classes ? kClasses : 1); ++c) {
      if (!b->cut_groups[c]) continue;
      const long long* cut = b->d_cut + b->cut_at[c];
      void* ba[] = {(void*)&b->d_segs, (void*)&b->nseg, (void*)&cut, (void*)&b->chunk};
      e = hipModuleLaunchKernel(b->classes ? b->f_class[c] : b->f_batch, (unsigned)b->cut_groups[c], 1, 1, 256, 1, 1, 0, s, ba,
                                nullptr);
      if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("batch kernel: ") + hipGetErrorString(e));
    }
    return QED_OK;
  }
  const unsigned groups = (unsigned)b->grid;
  if (!b->f_fix) {
    void* ba[] = {(void*)&b->d_segs, (void*)&b->d_share};
    e = hipModuleLaunchKernel(b->f_batch, groups, 1, 1, 256, 1, 1, 0, s, ba, nullptr);
    if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("batch kernel: ") + hipGetErrorString(e));
    return QED_OK;
  }
  void* zf[] = {(void*)&b->d_fix};
  e = hipModuleLaunchKernel(b->f_zero, 1, 1, 1, 64, 1, 1, 0, s, zf, nullptr);
  if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("zero kernel: ") + hipGetErrorString(e));
  unsigned* cnt = b->d_fix;
  unsigned* list = b->d_fix + 64;
  void* ba[] = {(void*)&b->d_segs, (void*)&b->d_share, (void*)&b->fix_kappa, (void*)&cnt, (void*)&list};
  e = hipModuleLaunchKernel(b->f_batch, groups, 1, 1, 256, 1, 1, 0, s, ba, nullptr);
  if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("batch kernel: ") + hipGetErrorString(e));
  void* fa[] = {(void*)&b->d_segs, (void*)&b->nseg, (void*)&cnt, (void*)&list};
  e = hipModuleLaunchKernel(b->f_fix, (unsigned)b->fix_grid, 1, 1, 256, 1, 1, 0, s, fa, nullptr);
  if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("fix-up kernel: ") + hipGetErrorString(e));
  return QED_OK;
}

// Adds `count` rounds of cost c each to waves of the given loads, one after the
// other to the wave with the least: take[w] rounds to wave w.  A level is searched that
// nearly all of them fill the waves to; the few left go to the lowest.
static void fill_waves(std::vector<double>& load, long long count, double c, std::vector<int>& take) {
  const size_t W = load.size();
  take.assign(W, 0);
  double lo = *std::min_element(load.begin(), load.end());
  double hi = *std::max_element(load.begin(), load.end()) + c * ((double)count / (double)W + 1);
  auto rounds = [&](double level, size_t w) { return level > load[w] ? (long long)((level - load[w]) / c) : 0LL; };
  auto total = [&](double level) {
    long long n = 0;
    for (size_t w = 0; w < W; ++w) n += rounds(level, w);
    return n;
  };
  while (hi - lo > 1e-3 * c && hi - lo > 1e-12 * hi) {
    const double mid = 0.5 * (lo + hi);
    (total(mid) <= count ? lo : hi) = mid;
  }
  long long left = count;
  for (size_t w = 0; w < W; ++w) {
    take[w] = (int)rounds(lo, w);
    left -= take[w];
    load[w] += take[w] * c;
  }
  std::vector<std::pair<double, size_t>> low(W);
  while (left > 0) {
    for (size_t w = 0; w < W; ++w) low[w] = {load[w], w};
    const size_t n = (size_t)std::min<long long>(left, (long long)W);
    std::nth_element(low.begin(), low.begin() + (n - 1), low.end());
    for (size_t i = 0; i < n; ++i) {
      ++take[low[i].second];
      load[low[i].second] += c;
    }
    left -= (long long)n;
  }
}

static qed_status layout_tiles(qed_batch_plan* b, const qed_segment* segs, const std::vector<int>& proc_of,
                               const std::vector<double>& cost) {
  // segments by decreasing cost per point, then tile offsets
  std::vector<int> ord(b->nseg);
  for (int i = 0; i < b->nseg; ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(), [&](int a, int c) { return cost[a] > cost[c]; });
  // (the pair module's classes come in that order)
  if (b->pair)
    std::stable_sort(ord.begin(), ord.end(),
                     [&](int a, int c) { return pair_class(segs[a].proc->n) < pair_class(segs[c].proc->n); });
  b->host.clear();
  long long t0 = 0, l0 = 0;
  int cls = 0;
  b->cls_tile[0] = 0;
  auto close_to = [&](int c) {
    for (; cls < c; ++cls) b->cls_tile[cls + 1] = t0;
  };
  std::vector<std::pair<long long, double>> tiles;  // end and cost per tile of every segment, in tile order
  for (int i : ord) {
    if (b->pair) close_to(pair_class(segs[i].proc->n));
    DevSeg d;
    d.mom = segs[i].momenta;
    d.hel = segs[i].hel;
    d.out = segs[i].out;
    d.N = segs[i].N;
    d.tile0 = t0;
    d.proc = b->pair ? segs[i].proc->n : proc_of[i];
    d.shift = b->shift[proc_of[i]];
    d.shift64 = b->shift64[proc_of[i]];
    d.list0 = l0;
    l0 += segs[i].N;
    b->host.push_back(d);
    const long long per = (64LL >> d.shift) * b->chunk;  // points per tile
    t0 += (segs[i].N + per - 1) / per;
    tiles.push_back({t0, tile_cost(cost[i])});
  }
  close_to(kClasses);
  b->ntiles = t0;
  if (b->pair) {
    std::vector<long long> cut;
    for (int c = 0; c < (b->classes ? kClasses : 1); ++c) {
      const long long lo = b->classes ? b->cls_tile[c] : 0, hi = b->classes ? b->cls_tile[c + 1] : t0;
      const long long most = b->classes ? (long long)b->ncu * kPairClasses[c].waves : b->ncu;
      const long long groups = std::min<long long>((hi - lo + 3) / 4, most);
      const long long W = 4 * groups;
      b->cut_at[c] = (int)cut.size();
      b->cut_groups[c] = (int)groups;
      if (!groups) continue;
      // wave w starts at the first tile with at least w / W of the cost before it
      double total = 0;
      long long t = lo;
      for (auto& g : tiles)
        if (g.first > t) {
          total += (double)(std::min(g.first, hi) - t) * g.second;
          t = std::max(t, std::min(g.first, hi));
        }
      double before = 0;
      t = lo;
      size_t g = 0;
      for (long long w = 0; w < W; ++w) {
        const double want = total * (double)w / (double)W;
        while (t < hi) {
          while (tiles[g].first <= t) ++g;
          if (before >= want - 1e-9 * total) break;
          const long long room = std::min(tiles[g].first, hi) - t;
          const long long n = std::min<long long>(room, std::max<long long>(1, (long long)((want - before) / tiles[g].second)));
          before += (double)n * tiles[g].second;
          t += n;
        }
        cut.push_back(t);
      }
      cut.push_back(hi);
    }
    hipError_t e = hipMemcpy(b->d_cut, cut.data(), sizeof(long long) * cut.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("tile ranges copy: ") + hipGetErrorString(e));
  }
  if (!b->pair && b->grid > 0) {
    // every wave the same cost: it takes some rounds of each segment, so that
    // errors of the cost model add up on none of them.  (Every W-th tile of W
    // waves gives some a tile of the dearest process more than others and
    // nothing for it: FP32C n = 1..6, 50001 points each, without the FP64 pass
    // 667 us, from a counter that waves take tiles from 573, these shares 560.)
    const size_t W = 4 * (size_t)b->grid;
    std::vector<double> load(W, 0.0);
    std::vector<int> take;
    std::vector<std::vector<int>> of(W);
    for (int k = 0; k < b->nseg; ++k) {
      const DevSeg& d = b->host[k];
      const long long per = 64LL >> d.shift, count = (d.N + per - 1) / per;
      if (!count) continue;
      fill_waves(load, count, cost[ord[k]] / (double)(1 << d.shift) + kLaneCost, take);
      long long first = 0;
      for (size_t w = 0; w < W; ++w)
        if (take[w]) {
          of[w].insert(of[w].end(), {k, (int)first, take[w]});
          first += take[w];
        }
    }
    std::vector<int> share(W + 1);
    for (size_t w = 0; w < W; ++w) {
      share[w] = (int)share.size();
      share.insert(share.end(), of[w].begin(), of[w].end());
    }
    share[W] = (int)share.size();
    hipError_t e = hipMemcpy(b->d_share, share.data(), sizeof(int) * share.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("wave shares copy: ") + hipGetErrorString(e));
  }
  hipError_t e = hipMemcpy(b->d_segs, b->host.data(), sizeof(DevSeg) * b->host.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("segment table copy: ") + hipGetErrorString(e));
  return QED_OK;
}

extern "C" qed_status qed_batch_plan_create(const qed_segment* segs, int nseg, int tile_points,
                                            qed_batch_plan** out) {
  if (!out) return fail(QED_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!segs || nseg <= 0 || nseg > 64) return fail(QED_ERR_INVALID_ARG, "need 1..64 segments");
  if (tile_points < 0 || tile_points % 64 || tile_points > 64 * 64)
    return fail(QED_ERR_INVALID_ARG, "tile_points must be 0 (autotune) or a multiple of 64 up to 4096");
  std::vector<const qed_process*> procs;
  std::vector<int> proc_of(nseg);
  std::vector<double> cost(nseg);
  for (int i = 0; i < nseg; ++i) {
    const qed_segment& s = segs[i];
    if (!s.proc) return fail(QED_ERR_INVALID_ARG, "segment " + std::to_string(i) + ": process is NULL");
    if (s.proc->mode != QED_HEL_PER_POINT)
      return fail(QED_ERR_UNSUPPORTED, "batches take per-point helicity processes");
    if (s.proc->n_in != 1) return fail(QED_ERR_UNSUPPORTED, "batches take one-incoming-photon processes");
    if (s.proc->prec != segs[0].proc->prec) return fail(QED_ERR_INVALID_ARG, "all processes must share precision");
    if (s.proc->var.fixup != segs[0].proc->var.fixup)
      return fail(QED_ERR_INVALID_ARG, "all processes must share the FP64 fix-up setting");
    if (s.N < 0) return fail(QED_ERR_INVALID_ARG, "segment " + std::to_string(i) + ": N < 0");
    if (s.N > 0 && (!s.momenta || !s.hel || !s.out))
      return fail(QED_ERR_INVALID_ARG, "segment " + std::to_string(i) + ": NULL buffer");
    if (s.N >= (1LL << 31)) return fail(QED_ERR_INVALID_ARG, "segment too large");
    // processes with the same kernel shape share one body in the module
    auto same = [&](const qed_process* q) {
      return q->var.subset == s.proc->var.subset &&
             variant_tag(q->var, q->proc.n_out, q->proc.n_in) == variant_tag(s.proc->var, s.proc->proc.n_out, s.proc->proc.n_in);
    };
    auto it = std::find_if(procs.begin(), procs.end(), same);
    if (it == procs.end()) {
      proc_of[i] = (int)procs.size();
      procs.push_back(s.proc);
    } else {
      proc_of[i] = (int)(it - procs.begin());
    }
    cost[i] = s.proc->info.flops_per_point;
  }
  auto b = std::make_unique<qed_batch_plan>();
  b->nseg = nseg;
  for (auto* p : procs) {
    const int graph = __builtin_ctz(cache_lanes(p->var));
    b->shift.push_back(pair_eval(p->proc, p->var) ? 1 : graph);
    b->shift64.push_back(pair_kernel(p->proc, p->var) ? 1 : graph);
  }
  // module (cached like every generated unit)
  std::string src;
  std::vector<std::pair<Process, Variant>> pv;
  for (auto* p : procs) pv.push_back({p->proc, batch_variant(p->var)});
  b->pair = all_pair(pv);
  try {
    src = b->pair ? pair_module_source() : module_source(pv);
  } catch (const std::exception& e) {
    return fail(QED_ERR_INVALID_ARG, std::string("batch emit: ") + e.what());
  }
  std::string tag = batch_tag(pv);
  std::string co;
  KernelMeta meta;
  bool hit;
  double ms;
  qed_status st = qedx_rt::get_code_object(tag, src, co, meta, hit, ms);
  if (st) return st;
  auto chk = [&](hipError_t e, const char* what) -> qed_status {
    if (e != hipSuccess) return fail(QED_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
    return QED_OK;
  };
  if ((st = chk(hipModuleLoadData(&b->mod, co.data()), "load batch module"))) return st;
  if ((st = chk(hipModuleGetFunction(&b->f_batch, b->mod, "qedx_batch"), "qedx_batch"))) return st;
  for (int c = 0; b->pair && c < kClasses; ++c)
    if ((st = chk(hipModuleGetFunction(&b->f_class[c], b->mod, kPairClasses[c].name), kPairClasses[c].name))) return st;
  if (hipMalloc((void**)&b->d_segs, sizeof(DevSeg) * nseg) != hipSuccess)
    return fail(QED_ERR_OOM, "segment table allocation failed");
  if (module_fixup(pv)) {
    long long total = 0;
    for (int i = 0; i < nseg; ++i) total += segs[i].N;
    if (total >= (1LL << 31)) return fail(QED_ERR_INVALID_ARG, "FP32C batches with the FP64 fix-up take < 2^31 points");
    if ((st = chk(hipModuleGetFunction(&b->f_zero, b->mod, "qedx_zero"), "qedx_zero"))) return st;
    if ((st = chk(hipModuleGetFunction(&b->f_fix, b->mod, "qedx_batch_fix"), "qedx_batch_fix"))) return st;
    if (hipMalloc((void**)&b->d_fix, sizeof(unsigned) * (64 + (size_t)std::max<long long>(total, 1))) != hipSuccess)
      return fail(QED_ERR_OOM, "fix-up list allocation failed");
    b->fix_kappa = segs[0].proc->info.fix_kappa;
    b->fix_grid = std::max<long long>(1, std::min<long long>((total + 255) / 256, 1024));
  }
  if ((st = chk(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking), "stream"))) return st;
  int dev = 0, ncu = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);

  b->ncu = ncu;
  // four waves per workgroup, up to four workgroups per compute unit
  if (b->pair && hipMalloc((void**)&b->d_cut, sizeof(long long) * ((size_t)16 * ncu + kClasses)) != hipSuccess)
    return fail(QED_ERR_OOM, "tile range allocation failed");
  if (!b->pair && hipMalloc((void**)&b->d_share, sizeof(int) * ((size_t)16 * ncu * (1 + 3 * (size_t)nseg) + 1)) != hipSuccess)
    return fail(QED_ERR_OOM, "wave share allocation failed");
  // plan signature for the autotune cache
  long long total_lanes = 0;
  for (int i = 0; i < nseg; ++i) total_lanes += segs[i].N << b->shift[proc_of[i]];
  std::ostringstream key;
  key << tag;
  for (int i = 0; i < nseg; ++i) key << "_" << segs[i].proc->n << "x" << segs[i].N;
  int grid = 0, chunk = 0;
  if (tile_points > 0) {
    chunk = tile_points / 64;
    grid = b->grid = ncu * 2;
    // one kernel per class where the batch fills the device several times over
    b->classes = b->pair && total_lanes >= (long long)ncu * 256 * 8;
  } else if (!tune_lookup(key.str(), grid, chunk)) {
    // time candidates: workgroups per CU (x 4 waves) and, for the pair module,
    // tile length (the others' shares are cut to single rounds).  The
    // inputs may still be in flight on another stream: wait for the device.
    if ((st = chk(hipDeviceSynchronize(), "autotune sync"))) return st;
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    // twice over all candidates, the better time of each: the first launches
    // after a pause run at a lower clock
    struct Candidate {
      int wpc, chunk;
      float ms;
    };
    std::vector<Candidate> cand;
    for (int wpc : {0, 1, 2, 4})  // 0: a kernel per class
      for (int ch : {1, 4, 16})
        if (b->pair ? wpc <= 1 && ch <= 4 : wpc > 0 && ch == 1) cand.push_back({wpc, ch, 1e30f});
    for (int pass = 0; pass < 2; ++pass)
      for (Candidate& c : cand) {
        b->classes = c.wpc == 0;
        b->grid = ncu * c.wpc;
        b->chunk = c.chunk;
        if ((st = layout_tiles(b.get(), segs, proc_of, cost))) return st;
        if ((st = launch_eager(b.get(), b->cap))) return st;  // warm
        (void)hipEventRecord(e0, b->cap);
        for (int r = 0; r < 3; ++r)
          if ((st = launch_eager(b.get(), b->cap))) return st;
        (void)hipEventRecord(e1, b->cap);
        if ((st = chk(hipEventSynchronize(e1), "autotune sync"))) return st;
        float t = 0;
        (void)hipEventElapsedTime(&t, e0, e1);
        c.ms = std::min(c.ms, t);
      }
    const Candidate& best = *std::min_element(cand.begin(), cand.end(), [](const Candidate& x, const Candidate& y) { return x.ms < y.ms; });
    grid = ncu * best.wpc;
    chunk = best.chunk;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    tune_store(key.str(), grid, chunk);
  }
  if (!tile_points) b->classes = b->pair && grid == 0;
  b->grid = grid;
  b->chunk = chunk;
  // (a grid from the cache of another device)
  if (!b->pair) b->grid = std::max(1, std::min(b->grid, 4 * ncu));
  if ((st = layout_tiles(b.get(), segs, proc_of, cost))) return st;
  // capture the kernels of a launch
  if ((st = chk(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal), "begin capture"))) return st;
  qed_status ls = launch_eager(b.get(), b->cap);
  hipError_t ce = hipStreamEndCapture(b->cap, &b->graph);
  if (ls) return ls;
  if ((st = chk(ce, "end capture"))) return st;
  if ((st = chk(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0), "instantiate"))) return st;
  *out = b.release();
  return QED_OK;
}

extern "C" qed_status qed_batch_launch(qed_batch_plan* plan, void* stream) {
  if (!plan) return fail(QED_ERR_INVALID_ARG, "plan is NULL");
  if (plan->ntiles == 0) return QED_OK;
  hipError_t e = hipGraphLaunch(plan->exec, (hipStream_t)stream);
  if (e != hipSuccess) return fail(QED_ERR_HIP, std::string("graph launch: ") + hipGetErrorString(e));
  return QED_OK;
}

extern "C" qed_status qed_batch_plan_destroy(qed_batch_plan* plan) {
  // launches may still be in flight on the caller's streams
  (void)hipDeviceSynchronize();
  delete plan;
  return QED_OK;
}

extern "C" qed_status qed_batch_info(const qed_batch_plan* plan, int64_t* ntiles, int* grid, int* chunk) {
  if (!plan) return fail(QED_ERR_INVALID_ARG, "plan is NULL");
  if (ntiles) *ntiles = plan->ntiles;
  if (grid) {
    // the workgroups that a launch starts, over all its kernels
    *grid = plan->pair ? 0 : plan->grid;
    for (int c = 0; plan->pair && c < (plan->classes ? kClasses : 1); ++c) *grid += plan->cut_groups[c];
  }
  if (chunk) *chunk = plan->chunk;
  return QED_OK;
}

// Ahead-of-time build of the batch module for processes n_list (per-point
// helicity, default kernel shapes) -- no GPU needed.
extern "C" qed_status qed_batch_prebuild(const int* n_list, int count, qed_precision prec, int rewrite,
                                          double* compile_ms) {
  if (rewrite < 0 || rewrite > 1) return fail(QED_ERR_INVALID_ARG, "rewrite must be 0 or 1");
  if (!n_list || count <= 0 || count > 64) return fail(QED_ERR_INVALID_ARG, "need 1..64 processes");
  std::vector<std::pair<Process, Variant>> pv;
  for (int i = 0; i < count; ++i) {
    int n = n_list[i];
    if (n < 1 || n > 6) return fail(QED_ERR_UNSUPPORTED, "n must be in 1..6");
    Variant v;
    qed_status st = qedx_rt::default_process_variant(n, QED_HEL_PER_POINT, prec, rewrite, v);
    if (st) return st;
    pv.push_back({Process::make(n, 1), batch_variant(v)});
  }
  std::string src;
  try {
    src = all_pair(pv) ? pair_module_source() : module_source(pv);
  } catch (const std::exception& e) {
    return fail(QED_ERR_INVALID_ARG, std::string("batch emit: ") + e.what());
  }
  std::string co;
  KernelMeta meta;
  bool hit;
  double ms = 0;
  qed_status st = qedx_rt::get_code_object(batch_tag(pv), src, co, meta, hit, ms);
  if (compile_ms) *compile_ms = ms;
  return st;
}
