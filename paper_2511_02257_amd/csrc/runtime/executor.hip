// Device runtime: leaf staging in pinned host memory, the arena borrowed from
// the caller, and execution of a placed plan on three HIP streams.
//
// Eager execution: per step s the spill stream copies the step's evicted
// intermediates to the host (D2H) and records ev_d2h[s]; the upload stream
// copies its missing operands in (H2D) and records ev_h2d[s]; the compute
// stream waits for the uploads of the step (and, where an output reuses
// memory a spill was still reading, for that spill), launches the step's
// kernels and records ev_comp[s].  A transfer into memory that kernels last
// touched at step k first waits for ev_comp[k]; an upload into memory a spill
// was reading, or of a tensor a spill wrote out, waits for that spill; a
// spill into host memory an upload was reading waits for that upload.  All
// waits come from the plan (place()), so uploads, spills and kernels overlap
// whenever the memory they use is already free.
// Time-slice passes (t_chunks > 1) repeat the plan on slices of every tensor,
// alternating between two halves of the memory; a pass waits for the one two
// before it (same half) to be done with that half.
// Graph replay: the same walk captured on one stream (segments of steps, the
// stream order carries every dependency), or added to one graph node by node
// with the walk's waits as explicit edges (no capture).  The eager walk can also be
// recorded instead of issued (trace_execute), so that its ordering can be
// checked on a host without a GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <cstdlib>
#include <thread>
#include <tuple>

#include "../ctx.hpp"
#include "../kernels/kernels.hpp"
#include "graph_order.hpp"
#include "walk.hpp"

namespace cdag {

namespace {
inline void ignore_last_error() { (void)hipGetLastError(); }
// A failed call also leaves its code as the thread's last error; it is read
// (and so cleared) here, or a later launch check would report it again.
void hip_check(hipError_t e, const char* what) {
  if (e != hipSuccess) {
    ignore_last_error();
    throw Error(CDAG_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
  }
}
#define HIPC(x) hip_check((x), #x)
inline void ignore(hipError_t) {}

double now() {
  return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// Most bytes of a step's transfers, in one direction, that are moved by a kernel
// where copies can run beside kernels (eager issue and the three-stream graph).
constexpr int64_t kKernelMoveBytes = 8 << 20;
}  // namespace

// ---------------------------------------------------------------- static scratch
// Device memory for cdag_execute_static, which allocates nothing: a fixed
// array that every GPU the library runs on holds until the process ends.  In
// host code `scratch` only names the symbol; its device address (one per GPU)
// comes from hipGetSymbolAddress when a context binds a device, and only that
// address is ever passed to kernels or copies.
constexpr int64_t kScratchBytes = CDAG_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {
std::mutex g_scratch_mu;
std::map<int, char*> g_scratch_ptr;   // device ordinal -> device address of `scratch`

// Called with `device` current; once per device.
void ensure_scratch_address(int device) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr.count(device)) return;
  void* ptr = nullptr;
  hip_check(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
  g_scratch_ptr[device] = static_cast<char*>(ptr);
}

char* scratch_address(int device) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  auto it = g_scratch_ptr.find(device);
  return it == g_scratch_ptr.end() ? nullptr : it->second;
}
}  // namespace

struct Device {
  int device = -1;
  hipStream_t comp = nullptr, copy = nullptr;   // borrowed: kernels, uploads
  hipStream_t spill_s = nullptr;                // owned: spills to the host
  char* arena = nullptr;
  uint64_t arena_bytes = 0;
  uint64_t arena_epoch = 0;                 // bumped when the arena is rebound
  // pinned staging of leaves in device layout, per precision mode
  std::vector<void*> stage[4];
  uint64_t stage_version[4] = {0, 0, 0, 0};
  // host spill pool: pinned, or pageable when a pinned allocation of the
  // plan's size fails (then steps run eagerly, without captured segments)
  void* spill = nullptr;
  int64_t spill_bytes = 0;
  bool spill_pageable = false;
  // pinned result buffer, written by the cross-sum kernel
  void* results = nullptr;
  int64_t results_bytes = 0;
  // per step of every pass and per stream role; then per pass, the pass-end
  // events of the three streams
  std::vector<hipEvent_t> ev[kStreams], ev_end[kStreams];
  hipEvent_t t0 = nullptr, t1 = nullptr;
  // what is currently uploaded
  uint64_t blob_key = 0, blob_epoch = 0;
  int resident_prec = -1;
  uint64_t resident_key = 0, resident_epoch = 0;
  // captured step sequence: one graph per segment of consecutive steps
  hipStream_t cap = nullptr;        // stream the one-stream segments are captured on
  hipEvent_t ev_join[2] = {nullptr, nullptr};
  std::vector<hipGraph_t> seg_graph;
  std::vector<hipGraphExec_t> seg_exec;
  uint64_t graph_key = 0, graph_epoch = 0, graph_stage = 0;
  int graph_mode = 0;
  void* graph_spill = nullptr;
  void* graph_results = nullptr;
  bool graph_finished = true;       // the last graph ends with the cross sums

  void drop_graphs() {
    for (auto g : seg_exec) ignore(hipGraphExecDestroy(g));
    for (auto g : seg_graph) ignore(hipGraphDestroy(g));
    seg_exec.clear();
    seg_graph.clear();
    graph_key = 0;
  }
  // timing mode: event pairs around kernel launches and host transfers
  std::vector<hipEvent_t> tpool;
  size_t tnext = 0;
  struct TPair {
    int64_t launch;          // launch index; -1: cross sum; -2: a transfer
    int32_t type, kinds;     // transfers: CDAG_LAUNCH_H2D / D2H and the tensor's kind bit
    int64_t step;
    double bytes;
    hipEvent_t a, b;
  };
  std::vector<TPair> tpairs;

  hipEvent_t timing_event() {
    if (tnext == tpool.size()) {
      hipEvent_t e;
      HIPC(hipEventCreate(&e));
      tpool.push_back(e);
    }
    return tpool[tnext++];
  }

  ~Device() {
    if (device >= 0) ignore(hipSetDevice(device));
    drop_graphs();
    if (cap) ignore(hipStreamDestroy(cap));
    if (spill_s) ignore(hipStreamDestroy(spill_s));
    for (int r = 0; r < kStreams; ++r) {
      for (auto e : ev[r]) ignore(hipEventDestroy(e));
      for (auto e : ev_end[r]) ignore(hipEventDestroy(e));
    }
    for (auto e : tpool) ignore(hipEventDestroy(e));
    if (t0) ignore(hipEventDestroy(t0));
    if (t1) ignore(hipEventDestroy(t1));
    for (auto e : ev_join)
      if (e) ignore(hipEventDestroy(e));
    for (auto& v : stage)
      for (void* p : v)
        if (p) ignore(hipHostFree(p));
    free_spill();
    if (results) ignore(hipHostFree(results));
  }
  void free_spill() {
    if (spill && spill_pageable) std::free(spill);
    else if (spill) ignore(hipHostFree(spill));
    spill = nullptr;
    spill_bytes = 0;
    spill_pageable = false;
  }
};

void device_destroy(Device* d) { delete d; }

void device_bind(Ctx& c, int device, void* compute_stream, void* copy_stream) {
  int n = 0;
  HIPC(hipGetDeviceCount(&n));
  if (device < 0 || device >= n) throw Error(CDAG_E_INVALID, "device ordinal out of range");
  if (!c.dev || c.dev->device != device) {
    delete c.dev;
    c.dev = nullptr;
    c.dev = new Device();
    c.dev->device = device;
  }
  HIPC(hipSetDevice(device));
  ensure_scratch_address(device);
  c.dev->comp = (hipStream_t)compute_stream;
  c.dev->copy = (hipStream_t)copy_stream;
  if (!c.dev->t0) {
    // library-owned streams keep the default priority
    HIPC(hipEventCreate(&c.dev->t0));
    HIPC(hipEventCreate(&c.dev->t1));
    for (auto& e : c.dev->ev_join) HIPC(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    HIPC(hipStreamCreateWithFlags(&c.dev->spill_s, hipStreamNonBlocking));
    HIPC(hipStreamCreateWithFlags(&c.dev->cap, hipStreamNonBlocking));
  }
}

void device_bind_arena(Ctx& c, void* arena, uint64_t bytes) {
  if (!c.dev) throw Error(CDAG_E_STATE, "cdag_bind_device first");
  c.dev->arena = (char*)arena;
  c.dev->arena_bytes = bytes;
  c.dev->arena_epoch++;
}

// Plan for (prec, batched) in the bound arena.
static void plan_for_arena(Ctx& c, int prec, int batched) { ensure_plan(c, prec, batched, c.dev->arena_bytes); }

namespace {
// Interleaved complex [nt][e] (S = double or float) -> planar [nt][2][e] in T.
template <typename S, typename T>
void to_device_layout(const S* src, T* dst, int64_t nt, int64_t e) {
  for (int64_t t = 0; t < nt; ++t) {
    const S* s = src + 2 * t * e;
    T* re = dst + 2 * t * e;
    T* im = re + e;
    for (int64_t i = 0; i < e; ++i) {
      re[i] = (T)s[2 * i];
      im[i] = (T)s[2 * i + 1];
    }
  }
}

void ensure_stage(Ctx& c, int prec) {
  Device& D = *c.dev;
  if (D.stage_version[prec] == c.data_version && !D.stage[prec].empty()) return;
  const int64_t L = c.dag.n_leaves;
  const int eb = prec == CDAG_FP64 ? 16 : 8;
  for (void* p : D.stage[prec])
    if (p) ignore(hipHostFree(p));
  D.stage[prec].assign(L, nullptr);
  for (int64_t u = 0; u < L; ++u)
    HIPC(hipHostMalloc(&D.stage[prec][u], (size_t)c.dag.size(u, eb), hipHostMallocDefault));
  const unsigned nth = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
  std::vector<std::thread> th;
  for (unsigned w = 0; w < nth; ++w)
    th.emplace_back([&, w] {
      for (int64_t u = w; u < L; u += nth) {
        const int64_t e = c.dag.elems(u) / c.dag.nt[u];
        const void* src = c.leaf_data[u].data();
        const bool c64 = c.leaf_dtype[u] == CDAG_C64;
        if (prec == CDAG_FP64) {
          if (c64) to_device_layout<float, double>((const float*)src, (double*)D.stage[prec][u], c.dag.nt[u], e);
          else to_device_layout<double, double>((const double*)src, (double*)D.stage[prec][u], c.dag.nt[u], e);
        } else {
          if (c64) to_device_layout<float, float>((const float*)src, (float*)D.stage[prec][u], c.dag.nt[u], e);
          else to_device_layout<double, float>((const double*)src, (float*)D.stage[prec][u], c.dag.nt[u], e);
        }
      }
    });
  for (auto& t : th) t.join();
  D.stage_version[prec] = c.data_version;
}

void ensure_events(Device& D, size_t steps, size_t passes) {
  for (int r = 0; r < kStreams; ++r) {
    for (auto* v : {&D.ev[r], &D.ev_end[r]}) {
      const size_t n = v == &D.ev[r] ? steps : passes;
      while (v->size() < n) {
        hipEvent_t e;
        HIPC(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        v->push_back(e);
      }
    }
  }
}

// The spill pool holds the plan's spilled intermediates at once.  Pinned
// memory of that size may be refused; pageable memory then takes its place.
void ensure_spill(Device& D, int64_t need_bytes) {
  if (D.spill && D.spill_bytes >= need_bytes) return;
  D.free_spill();
  if (need_bytes <= 0) return;
  if (hipHostMalloc(&D.spill, (size_t)need_bytes, hipHostMallocDefault) != hipSuccess) {
    ignore_last_error();
    D.spill = std::malloc((size_t)need_bytes);
    if (!D.spill) throw Error(CDAG_E_NOMEM, "host spill pool of " + std::to_string(need_bytes) + " bytes");
    D.spill_pageable = true;
  }
  D.spill_bytes = need_bytes;
}

// Coherent, so that what a kernel stored there is seen by the host once the
// stream has been waited for.
void ensure_pinned(void*& p, int64_t& have, int64_t need_bytes) {
  if (have >= need_bytes && p) return;
  if (p) ignore(hipHostFree(p));
  p = nullptr;
  have = 0;
  if (need_bytes <= 0) return;
  HIPC(hipHostMalloc(&p, (size_t)need_bytes, hipHostMallocMapped | hipHostMallocCoherent));
  have = need_bytes;
}

hipError_t call_of(const Launch& L, int prec, char* arena, KernelCall* k) {
  switch (L.type) {
    case L_HEC:
      return hec_call(prec, L.tile, L.interior != 0, arena, L.desc_off, L.n_desc, L.n_items, k, L.tr_desc_off,
                      L.tr_n_desc, L.tr_n_items);
    case L_RED: return reduce_call(prec, arena, L.desc_off, L.n_desc, L.n_items, k);
    case L_HCA: return hca_call(prec, arena, L.desc_off, L.n_desc, L.n_items, k);
    default: throw Error(CDAG_E_STATE, "bad launch type");
  }
}

// The last kernel of an execute: the cross sums, and the results to `host`.
hipError_t finish_call(const KernelPlan& kp, char* arena, char* host, KernelCall* k) {
  return xsum_call(arena, kp.xsum.desc_off, kp.xsum_entries_off, kp.xsum.n_desc, kp.xsum.n_items, kp.corr_off,
                   kp.corr_bytes, host, k);
}

hipError_t launch_finish(const KernelPlan& kp, char* arena, char* host, hipStream_t st) {
  KernelCall k;
  const hipError_t e = finish_call(kp, arena, host, &k);
  return e != hipSuccess ? e : launch(k, st);
}

hipError_t launch_one(const Launch& L, int prec, char* arena, hipStream_t st) {
  KernelCall k;
  const hipError_t e = call_of(L, prec, arena, &k);
  return e != hipSuccess ? e : launch(k, st);
}

// Kernels of global step g; with `timed`, every launch is bracketed by an
// event pair.
int64_t launch_step(const KernelPlan& kp, int64_t g, int prec, char* arena, hipStream_t st, Device* timed) {
  int64_t n = 0;
  for (int64_t li = kp.launch_off[g]; li < kp.launch_off[g + 1]; ++li) {
    const Launch& L = kp.launches[li];
    if (timed) {
      hipEvent_t a = timed->timing_event(), b = timed->timing_event();
      HIPC(hipEventRecord(a, st));
      HIPC(launch_one(L, prec, arena, st));
      HIPC(hipEventRecord(b, st));
      timed->tpairs.push_back({li, 0, 0, g, 0.0, a, b});
    } else {
      HIPC(launch_one(L, prec, arena, st));
    }
    ++n;
  }
  return n;
}

// Ends of one transfer of pass m: an upload from the leaf's staging or the
// spill pool, or a spill.
Move move_of(const Ctx& c, const Device& D, int prec, const PlanRec& r, const PassMap& m) {
  char* spill = (char*)D.spill;
  char* dev = D.arena + m.dev(r.dev_off);
  if (r.op == OP_D2H) return {dev, spill + m.host(r.host_off), m.bytes(r.node)};
  const void* src = c.dag.is_leaf(r.node) ? (const void*)((const char*)D.stage[prec][r.node] + m.stage(r.node))
                                          : (const void*)(spill + m.host(r.host_off));
  return {src, dev, m.bytes(r.node)};
}

// The issuing form: kernels on st[S_COMP], uploads on st[S_H2D], spills on
// st[S_D2H], with the device's per-step and per-pass events.
struct HipOps {
  const Ctx& c;
  Device& D;
  int prec;
  hipStream_t st[kStreams];
  Device* timed;

  std::vector<Move> moves[kStreams]{};   // of the step, not yet issued

  void wait(int to, int from, int64_t g, int64_t) { HIPC(hipStreamWaitEvent(st[to], D.ev[from][g], 0)); }
  void record(int r, int64_t g) {   // comes after the step's transfers on r
    flush(r);
    HIPC(hipEventRecord(D.ev[r][g], st[r]));
  }
  void wait_pass(int to, int from, int64_t k, int64_t) { HIPC(hipStreamWaitEvent(st[to], D.ev_end[from][k], 0)); }
  void record_pass(int r, int64_t k, int64_t) { HIPC(hipEventRecord(D.ev_end[r][k], st[r])); }
  int64_t launch(int64_t g, const PassMap&) { return launch_step(c.kplan, g, prec, D.arena, st[S_COMP], timed); }
  void copy(int r, const Move& mv) {
    HIPC(hipMemcpyAsync(mv.dst, mv.src, (size_t)mv.bytes, r == S_D2H ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice,
                        st[r]));
  }
  // Small transfers of a step go in one launch (a copy costs 5 to 10 us of its
  // own on a stream: a pass with 4 leaves of 32 KiB 113 -> 86 us, one with 12 of
  // 680 KB 1.13 -> 1.00 ms); large ones to the copy engines, which leave the
  // compute units to the kernels (leaves of 17 MB a pass).
  void flush(int r) {
    int64_t bytes = 0;
    for (const Move& mv : moves[r]) bytes += mv.bytes;
    if (bytes <= kKernelMoveBytes && !(D.spill_pageable && D.spill)) {
      HIPC(launch_moves(moves[r].data(), (int)moves[r].size(), st[r]));
    } else {
      for (const Move& mv : moves[r]) copy(r, mv);
    }
    moves[r].clear();
  }
  void transfer(const PlanRec& r, const PassMap& m, int64_t g) {
    const Move mv = move_of(c, D, prec, r, m);
    const int role = r.op == OP_D2H ? S_D2H : S_H2D;
    if (!timed) {
      moves[role].push_back(mv);
      return;
    }
    hipEvent_t ta = timed->timing_event(), tb = timed->timing_event();
    HIPC(hipEventRecord(ta, st[role]));
    copy(role, mv);
    HIPC(hipEventRecord(tb, st[role]));
    const int32_t kd = c.dag.kind[r.node];
    timed->tpairs.push_back({-2, r.op == OP_D2H ? CDAG_LAUNCH_D2H : CDAG_LAUNCH_H2D,
                             kd >= 0 ? (1 << kd) : 0, g, (double)mv.bytes, ta, tb});
  }
};

// The one-stream form that segments are captured with: stream order carries
// every dependency, and the spills, then the uploads, of a step are one launch
// each.
struct SegmentOps {
  const Ctx& c;
  Device& D;
  int prec;
  hipStream_t st;
  std::vector<Move> moves{};
  int32_t dir = OP_D2H;

  void wait(int, int, int64_t, int64_t) {}
  void record(int, int64_t) {}
  void wait_pass(int, int, int64_t, int64_t) {}
  void record_pass(int, int64_t, int64_t) {}
  void flush() {
    if (!moves.empty()) HIPC(launch_moves(moves.data(), (int)moves.size(), st));
    moves.clear();
  }
  void transfer(const PlanRec& r, const PassMap& m, int64_t) {
    if (r.op != dir) flush();
    dir = r.op;
    moves.push_back(move_of(c, D, prec, r, m));
  }
  int64_t launch(int64_t g, const PassMap&) {
    flush();
    return launch_step(c.kplan, g, prec, D.arena, st, nullptr);
  }
};

// The recording form: the same walk with no HIP call, writing what each stream
// would do (event records and waits, and the byte ranges that every transfer
// and every step's kernels read and write).  Event ids: kStreams * g + stream
// for the step events, kStreams * (passes * S + k) + stream for the pass-end
// events.  fail_at >= 0 throws at that record, as a failed HIP call would.
struct TraceOps {
  const Ctx& c;
  int prec;
  std::vector<cdag_trace_rec>& out;
  int64_t fail_at;
  int64_t seq = 0;

  void put(const cdag_trace_rec& r) {
    if ((int64_t)out.size() == fail_at)
      throw Error(CDAG_E_HIP, "injected failure at trace record " + std::to_string(fail_at));
    out.push_back(r);
  }
  static cdag_trace_rec blank(int32_t op, int32_t stream, int64_t step) {
    cdag_trace_rec r{};
    r.op = op;
    r.stream = stream;
    r.step = step;
    r.seq = r.node = r.event = -1;
    return r;
  }
  int64_t pass_event(int64_t k, int r) const {
    return kStreams * (std::max(c.plan.n_xsteps(), c.plan.chunks() * (int64_t)c.plan.steps.size()) + k) + r;
  }
  void event(int32_t op, int32_t stream, int64_t id, int64_t g) {
    cdag_trace_rec r = blank(op, stream, g);
    r.event = id;
    put(r);
  }
  void access(int32_t op, int32_t stream, int64_t g, int64_t node, int32_t space, int64_t off, int64_t bytes) {
    cdag_trace_rec r = blank(op, stream, g);
    r.seq = seq;
    r.node = node;
    r.space = space;
    r.off = off;
    r.bytes = bytes;
    put(r);
  }
  void wait(int to, int from, int64_t ev_g, int64_t g) { event(CDAG_TR_WAIT, to, kStreams * ev_g + from, g); }
  void record(int r, int64_t g) { event(CDAG_TR_RECORD, r, kStreams * g + r, g); }
  void wait_pass(int to, int from, int64_t k, int64_t g) { event(CDAG_TR_WAIT, to, pass_event(k, from), g); }
  void record_pass(int r, int64_t k, int64_t g) { event(CDAG_TR_RECORD, r, pass_event(k, r), g); }
  void transfer(const PlanRec& r, const PassMap& m, int64_t) {
    const int64_t bytes = m.bytes(r.node), g = m.k * (int64_t)c.plan.steps.size() + r.step;   // its plan step
    if (r.op == OP_D2H) {
      access(CDAG_TR_READ, S_D2H, g, r.node, CDAG_SPACE_ARENA, m.dev(r.dev_off), bytes);
      access(CDAG_TR_WRITE, S_D2H, g, r.node, CDAG_SPACE_SPILL, m.host(r.host_off), bytes);
    } else {
      if (c.dag.is_leaf(r.node)) access(CDAG_TR_READ, S_H2D, g, r.node, CDAG_SPACE_STAGE, m.stage(r.node), bytes);
      else access(CDAG_TR_READ, S_H2D, g, r.node, CDAG_SPACE_SPILL, m.host(r.host_off), bytes);
      access(CDAG_TR_WRITE, S_H2D, g, r.node, CDAG_SPACE_ARENA, m.dev(r.dev_off), bytes);
    }
    ++seq;
  }
  int64_t launch(int64_t g, const PassMap& m) {
    const Plan& p = c.plan;
    const Plan::Program& prog = p.program(m.k);
    const int64_t s = g - p.xfirst(m.k);
    for (int64_t ri = prog.off[s]; ri < prog.off[s + 1]; ++ri) {
      const PlanRec& r = prog.recs[ri];
      if (r.op != OP_EXEC) continue;
      const int64_t* ch = c.dag.children_begin(r.node);
      access(CDAG_TR_READ, S_COMP, g, ch[0], CDAG_SPACE_ARENA, m.operand(ch[0], r.a_off), m.bytes(ch[0]));
      access(CDAG_TR_READ, S_COMP, g, ch[1], CDAG_SPACE_ARENA, m.operand(ch[1], r.b_off), m.bytes(ch[1]));
      if (c.dag.kind[r.node] != HCA)
        access(CDAG_TR_WRITE, S_COMP, g, r.node, CDAG_SPACE_ARENA, m.dev(r.dev_off), m.bytes(r.node));
    }
    ++seq;
    return c.kplan.launch_off[g + 1] - c.kplan.launch_off[g];
  }
};

// The graph form: the same walk adding the transfers and kernels to a HIP
// graph as nodes with explicit dependencies (no stream capture), which
// GraphOrder works out: kernels, and a step's small transfers (moved by a
// kernel), are one chain; large transfers are copy nodes beside it.
struct GraphOps {
  const Ctx& c;
  Device& D;
  int prec;
  hipGraph_t graph;
  GraphOrder<hipGraphNode_t> order;
  std::vector<hipGraphNode_t> deps;
  std::vector<Move> moves[kStreams];                 // of the step, not yet added

  GraphOps(const Ctx& ctx, Device& dev, int p, hipGraph_t g)
      : c(ctx), D(dev), prec(p), graph(g), order(ctx.plan.n_xsteps(), ctx.plan.chunks()) {}
  void wait(int to, int from, int64_t g, int64_t) { order.wait(to, from, g); }
  void record(int r, int64_t g) {   // comes after the step's transfers on r
    flush(r);
    order.record(r, g);
  }
  void wait_pass(int to, int from, int64_t k, int64_t) { order.wait_pass(to, from, k); }
  void record_pass(int r, int64_t k, int64_t) { order.record_pass(r, k); }
  void transfer(const PlanRec& r, const PassMap& m, int64_t) {
    moves[r.op == OP_D2H ? S_D2H : S_H2D].push_back(move_of(c, D, prec, r, m));
  }
  // Small transfers of the step on stream r go into the chain, one kernel node
  // per kMaxMoves; large ones are copy nodes beside it (headline in 8 passes:
  // 57 ms, as kernels 65).
  void flush(int r) {
    int64_t bytes = 0;
    for (const Move& mv : moves[r]) bytes += mv.bytes;
    if (bytes > kKernelMoveBytes) {
      for (const Move& mv : moves[r]) {
        order.deps_of(r, false, &deps);
        hipGraphNode_t n = nullptr;
        HIPC(hipGraphAddMemcpyNode1D(&n, graph, deps.data(), deps.size(), mv.dst, mv.src, (size_t)mv.bytes,
                                     r == S_D2H ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice));
        order.added(r, false, n);
      }
      moves[r].clear();
      return;
    }
    for (size_t done = 0; done < moves[r].size();) {
      MoveBatch mb;
      const int k = make_moves(moves[r].data() + done, (int)(moves[r].size() - done), &mb);
      if (k <= 0) throw Error(CDAG_E_INVALID, "transfer too large");
      void* args[1] = {&mb};
      if (mb.begin[k] > 0) add_kernel(r, move_fn(), (unsigned)mb.begin[k], 256, args);
      done += (size_t)k;
    }
    moves[r].clear();
  }
  void add_kernel(int r, const void* fn, unsigned grid, unsigned block, void** args) {
    hipKernelNodeParams np{};
    np.func = const_cast<void*>(fn);
    np.gridDim = dim3(grid);
    np.blockDim = dim3(block);
    np.sharedMemBytes = 0;
    np.kernelParams = args;
    np.extra = nullptr;
    order.deps_of(r, true, &deps);
    hipGraphNode_t n = nullptr;
    HIPC(hipGraphAddKernelNode(&n, graph, deps.data(), deps.size(), &np));
    order.added(r, true, n);
  }
  void kernel(KernelCall& k) {
    k.bind();
    add_kernel(S_COMP, k.fn, k.grid, k.block, k.args);
  }
  int64_t launch(int64_t g, const PassMap&) {
    const KernelPlan& kp = c.kplan;
    for (int64_t li = kp.launch_off[g]; li < kp.launch_off[g + 1]; ++li) {
      KernelCall k;
      HIPC(call_of(kp.launches[li], prec, D.arena, &k));
      kernel(k);
    }
    return kp.launch_off[g + 1] - kp.launch_off[g];
  }
  // The cross sums end a graph that is one chain; with copy nodes beside it
  // they are launched after the graph.
  void finish() {
    if (order.copies()) return;
    KernelCall k;
    HIPC(finish_call(c.kplan, D.arena, (char*)D.results, &k));
    kernel(k);
  }
};

constexpr int64_t kSegmentSteps = 64;   // steps per one-stream graph when transfers are present
}  // namespace

// Autotuner: for every distinct (kind, N) among the exterior contractions,
// time each kernel choice, and what runs without one, on a synthetic
// contraction of that shape (operands in the arena's tensor pool, which holds
// nothing between executes).  uniform = false keeps the fastest per time slice
// of each shape; uniform = true keeps the one choice whose time over the whole
// DAG (per-slice time x the slices of that shape in the DAG, summed over
// shapes) is least, so that every wave runs its exterior contractions in one
// grouped launch.  The choices enter the tile table of the context
// (store_choices()).
int64_t device_autotune(Ctx& c, int prec, int batched, int reps, bool uniform) {
  Device& D = *c.dev;
  HIPC(hipSetDevice(D.device));
  if (!D.arena) throw Error(CDAG_E_STATE, "cdag_bind_arena first");
  plan_for_arena(c, prec, batched);
  const Plan& p = c.plan;
  const KernelPlan& kp = c.kplan;
  if ((uint64_t)kp.total_bytes > D.arena_bytes) throw Error(CDAG_E_NOMEM, "arena smaller than the plan");
  (void)batched;
  const int64_t eb = prec == CDAG_FP64 ? 16 : 8, acc = prec == CDAG_FP64 ? 8 : 4;
  auto al = [](int64_t x) { return (x + 255) / 256 * 256; };
  const int64_t lo = al(p.leaf_region_bytes), hi = kp.ws_off + kp.ws_bytes;
  // without resident leaves the synthetic operands lie where a resident plan
  // keeps its leaves, so its next execute uploads them again
  if (!c.leaves_resident) D.resident_prec = -1;
  const auto shapes = tune_shapes(c.dag);
  std::map<std::pair<int, int>, TuneRow> rows;   // time per slice, per candidate
  for (const auto& sh : shapes) rows[sh.first].weight = 0.0;
  // slices of each shape in the DAG (the uniform choice's weights)
  for (int64_t u = c.dag.n_leaves; u < c.dag.n_nodes(); ++u) {
    const auto row = rows.find({c.dag.kind[u], c.dag.nvec[u]});
    if (row != rows.end()) row->second.weight += c.dag.nt[u];
  }
  hipEvent_t e0, e1;
  HIPC(hipEventCreate(&e0));
  HIPC(hipEventCreate(&e1));
  try {
    for (const auto& sh : shapes) {
      const int kind = sh.first.first, n = sh.first.second, snt = sh.second.nt;
      TuneRow& row = rows[sh.first];
      for (int ch = 0; ch <= kNoChoice; ++ch) {
        HecDesc h{};
        // split count of a real contraction
        const int v = decompose_candidate(sh.second.gemm, snt, ch, prec, kind, n, &h);
        if (ch == kNoChoice) {
          row.default_variant = v;
        } else if (!choice_split_k(ch)) {
          HecDesc a{};
          decompose(sh.second.gemm, snt, v, prec, &a);
          if (a.splits == 1) {                          // same work items as the split choice
            row.t[ch] = row.t[choice_of(v, true)];
            continue;
          }
        }
        const int64_t slice_items = (int64_t)h.tiles_m * h.tiles_n * h.splits;
        const int64_t slice = (int64_t)h.M * h.K * eb + (int64_t)h.K * h.N * eb + (int64_t)h.M * h.N * eb;
        const int64_t wslice = h.splits > 1 ? (int64_t)h.splits * 2 * h.M * h.N * acc : 0;
        // A wave holds many contractions of one shape: time a batch of slices
        // with at least 4096 work items (at most 64 contractions' worth).
        int64_t want = std::max<int64_t>(snt, (4096 + slice_items - 1) / slice_items);
        want = std::min<int64_t>(want, 64LL * snt);
        int64_t nt = std::min<int64_t>(want, (hi - lo - 4096) / std::max<int64_t>(1, slice + wslice + 1024));
        if (nt < 1 || nt * slice_items > INT32_MAX) continue;
        h.nt = (int32_t)nt;
        h.tile_count = (int32_t)(nt * slice_items);
        const int64_t a = lo, b = a + al(nt * h.M * h.K * eb), cc = b + al(nt * h.K * h.N * eb);
        const int64_t ws = cc + al(nt * h.M * h.N * eb);
        const int64_t ws_bytes = h.splits > 1 ? al((int64_t)h.splits * nt * 2 * h.M * h.N * acc) : 0;
        const int64_t desc = ws + ws_bytes;
        if (desc + 256 > hi) continue;
        h.a_off = a;
        h.b_off = b;
        h.c_off = cc;
        h.ws_off = h.splits > 1 ? ws : -1;
        h.tile_begin = 0;
        RedDesc r{ws, cc, h.M * h.N, (int32_t)nt, h.splits, 0};
        const int64_t n_red = red_items(nt, (int64_t)h.M * h.N);
        HIPC(hipMemsetAsync(D.arena + a, 0, (size_t)(ws - a), D.comp));
        HIPC(hipMemcpyAsync(D.arena + desc, &h, sizeof(h), hipMemcpyHostToDevice, D.comp));
        HIPC(hipMemcpyAsync(D.arena + desc + 128, &r, sizeof(r), hipMemcpyHostToDevice, D.comp));
        const bool interior =
            hec_interior(h, kTileShapes[variant_tile(v)].bm, kTileShapes[variant_tile(v)].bn, k_step(prec));
        auto once = [&] {
          HIPC(launch_hec(prec, v, interior, D.arena, desc, 1, h.tile_count, D.comp));
          if (h.splits > 1) HIPC(launch_reduce(prec, D.arena, desc + 128, 1, n_red, D.comp));
        };
        once();
        HIPC(hipEventRecord(e0, D.comp));
        for (int k = 0; k < reps; ++k) once();
        HIPC(hipEventRecord(e1, D.comp));
        HIPC(hipEventSynchronize(e1));
        float ms = 0;
        HIPC(hipEventElapsedTime(&ms, e0, e1));
        row.t[ch] = ms / reps / (double)nt;
      }
    }
  } catch (...) {
    ignore(hipEventDestroy(e0));
    ignore(hipEventDestroy(e1));
    throw;
  }
  ignore(hipEventDestroy(e0));
  ignore(hipEventDestroy(e1));
  HIPC(hipStreamSynchronize(D.comp));
  return store_choices(rows, prec, uniform, &c.tiles);
}

// In-situ autotuner: for every distinct (kind, N) in turn, run the planned DAG
// `reps` times with each kernel choice, and without one, for that shape (the
// other shapes keep their current choice), with HIP events around every
// launch, and keep the one whose fastest execute spends the least time in
// exterior contractions plus split-K reductions.
int64_t device_autotune_insitu(Ctx& c, int prec, int batched, int reps) {
  const auto shapes = tune_shapes(c.dag);
  const bool timing = c.timing;
  const auto tiles = c.tiles;                  // restored if a trial execute throws
  c.timing = true;
  int64_t tuned = 0;
  try {
    for (const auto& sh : shapes) {
      const auto key = std::make_tuple(prec, sh.first.first, sh.first.second);
      TuneRow row;
      for (int v = 0; v <= kNoChoice; ++v) {
        if (v < kNumChoices && !choice_split_k(v)) {
          // the no-split setting only differs where the rule would split
          HecDesc h{};
          decompose(sh.second.gemm, sh.second.nt, choice_variant(v), prec, &h);
          if (h.splits == 1) continue;
        }
        if (v == kNoChoice) c.tiles.erase(key);
        else c.tiles[key] = v;
        c.version++;
        plan_for_arena(c, prec, batched);
        if ((uint64_t)c.kplan.total_bytes > c.dev->arena_bytes) continue;
        double t = 1e300;                        // fastest of the reps (robust to noise)
        for (int r = 0; r < reps; ++r) {
          cdag_exec_stats st{};
          device_execute(c, prec, batched, &st);
          double tr = 0;
          for (const cdag_launch_record& rec : c.records)
            if (rec.type == CDAG_LAUNCH_HEC || rec.type == CDAG_LAUNCH_REDUCE) tr += rec.ms;
          t = std::min(t, tr);
        }
        row.t[v] = t;
      }
      c.tiles.erase(key);                        // where not one of them fits the arena
      tuned += store_choices({{sh.first, row}}, prec, false, &c.tiles);
      c.version++;
    }
  } catch (...) {
    c.timing = timing;
    c.tiles = tiles;
    c.version++;
    throw;
  }
  c.timing = timing;
  return tuned;
}

void trace_execute(const Ctx& c, int prec, std::vector<cdag_trace_rec>& out, int64_t fail_at) {
  out.clear();
  TraceOps ops{c, prec, out, fail_at};
  walk_steps(c, 0, c.plan.n_xsteps(), false, false, ops);
}

namespace {
// Capture global steps [g0, g1) into one graph on one stream (stream order
// carries every dependency); the last segment ends with the cross sums.
hipGraph_t capture_steps(Ctx& c, Device& D, int prec, int64_t g0, int64_t g1, bool last) {
  hipGraph_t g = nullptr;
  HIPC(hipStreamBeginCapture(D.cap, hipStreamCaptureModeThreadLocal));
  try {
    SegmentOps ops{c, D, prec, D.cap};
    walk_steps(c, g0, g1, true, true, ops);
    if (last) HIPC(launch_finish(c.kplan, D.arena, (char*)D.results, D.cap));
  } catch (...) {
    ignore(hipStreamEndCapture(D.cap, &g));
    if (g) ignore(hipGraphDestroy(g));
    throw;
  }
  HIPC(hipStreamEndCapture(D.cap, &g));
  return g;
}

// Build the whole step sequence as one graph over the three streams' work,
// with the plan's waits as explicit edges.  *finished: whether it ends with the
// cross sums.
hipGraph_t build_graph(Ctx& c, Device& D, int prec, bool* finished) {
  hipGraph_t g = nullptr;
  HIPC(hipGraphCreate(&g, 0));
  try {
    GraphOps ops(c, D, prec, g);
    walk_steps(c, 0, c.plan.n_xsteps(), false, false, ops);
    ops.finish();
    *finished = !ops.order.copies();
  } catch (...) {
    ignore(hipGraphDestroy(g));
    throw;
  }
  return g;
}
}  // namespace

void device_execute(Ctx& c, int prec, int batched, cdag_exec_stats* st) {
  Device& D = *c.dev;
  const double tw0 = now();
  HIPC(hipSetDevice(D.device));
  if (D.arena) plan_for_arena(c, prec, batched);
  const Plan& p = c.plan;
  const KernelPlan& kp = c.kplan;
  if (!D.arena) throw Error(CDAG_E_STATE, "cdag_bind_arena first");
  if ((uint64_t)kp.total_bytes > D.arena_bytes)
    throw Error(CDAG_E_NOMEM, "arena has " + std::to_string(D.arena_bytes) + " bytes, the plan needs " +
                                  std::to_string(kp.total_bytes));
  const int eb = prec == CDAG_FP64 ? 16 : 8;
  ensure_stage(c, prec);
  ensure_spill(D, p.halves() * p.host_spill_bytes);
  ensure_pinned(D.results, D.results_bytes, kp.corr_bytes + kp.sums_bytes);
  const int64_t G = p.n_xsteps();
  ensure_events(D, (size_t)std::max<int64_t>(G, 1), (size_t)p.chunks());

  // descriptor tables: one upload per (plan, arena)
  const uint64_t pkey = c.plan_serial;
  if (D.blob_key != pkey || D.blob_epoch != D.arena_epoch) {
    HIPC(hipMemcpyAsync(D.arena + kp.blob_off, kp.blob.data(), kp.blob.size(), hipMemcpyHostToDevice, D.comp));
    HIPC(hipStreamSynchronize(D.comp));
    D.blob_key = pkey;
    D.blob_epoch = D.arena_epoch;
  }
  // leaves kept resident in their own region: one upload per (precision, arena, build)
  if (c.leaves_resident &&
      (D.resident_prec != prec || D.resident_epoch != D.arena_epoch || D.resident_key != D.stage_version[prec])) {
    D.resident_prec = -1;                        // until every leaf is there
    for (int64_t u = 0; u < c.dag.n_leaves; ++u)
      HIPC(hipMemcpyAsync(D.arena + p.leaf_off[u], D.stage[prec][u], (size_t)c.dag.size(u, eb),
                          hipMemcpyHostToDevice, D.copy));
    HIPC(hipStreamSynchronize(D.copy));
    D.resident_prec = prec;
    D.resident_epoch = D.arena_epoch;
    D.resident_key = D.stage_version[prec];
  }
  // a plan with the leaves on the host keeps its own tensors where a resident
  // plan keeps the leaves, so the next resident execute uploads them again
  if (!c.leaves_resident) D.resident_prec = -1;

  bool has_copies = false;
  for (const PlanRec& r : p.recs)
    if (r.op == OP_H2D || r.op == OP_D2H) { has_copies = true; break; }

  int64_t n_launch = 0, n_segments = 0;
  D.tnext = 0;
  D.tpairs.clear();
  Device* timed = c.timing ? &D : nullptr;
  const bool graphs = c.use_graphs && !c.timing && !D.spill_pageable;
  HIPC(hipEventRecord(D.t0, D.comp));
  if (graphs) {
    // replay graphs: one-stream segments of kSegmentSteps steps when there are
    // transfers (else one), or one graph built over the three streams; the
    // cross sums are the last one's last node where it has no copy nodes
    // (launched after the graphs they started 23 us after the last kernels)
    const bool one = c.use_graphs == 1;
    const int64_t seg = one && has_copies ? kSegmentSteps : std::max<int64_t>(G, 1);
    if (D.graph_key != pkey || D.graph_epoch != D.arena_epoch || D.graph_spill != D.spill ||
        D.graph_stage != D.stage_version[prec] || D.graph_mode != c.use_graphs || D.graph_results != D.results) {
      D.drop_graphs();
      D.graph_finished = true;
      for (int64_t g0 = 0; g0 == 0 || g0 < G; g0 += seg) {
        hipGraph_t g = nullptr;
        try {
          g = one ? capture_steps(c, D, prec, g0, std::min(G, g0 + seg), g0 + seg >= G)
                  : build_graph(c, D, prec, &D.graph_finished);
        } catch (...) {
          D.drop_graphs();
          throw;
        }
        D.seg_graph.push_back(g);
        hipGraphExec_t ge = nullptr;
        HIPC(hipGraphInstantiate(&ge, g, nullptr, nullptr, 0));
        D.seg_exec.push_back(ge);
      }
      D.graph_key = pkey;
      D.graph_epoch = D.arena_epoch;
      D.graph_spill = D.spill;
      D.graph_results = D.results;
      D.graph_stage = D.stage_version[prec];
      D.graph_mode = c.use_graphs;
    }
    for (hipGraphExec_t ge : D.seg_exec) HIPC(hipGraphLaunch(ge, D.comp));
    if (!D.graph_finished) HIPC(launch_finish(kp, D.arena, (char*)D.results, D.comp));
    n_segments = (int64_t)D.seg_exec.size();
    for (int64_t g = 0; g < G; ++g) n_launch += kp.launch_off[g + 1] - kp.launch_off[g];
  } else {
    HipOps ops{c, D, prec, {D.comp, D.copy, D.spill_s}, timed, {}};
    n_launch += walk_steps(c, 0, G, false, false, ops);
    // the cross sums, and the caller's later work, follow every transfer
    HIPC(hipEventRecord(D.ev_join[0], D.copy));
    HIPC(hipEventRecord(D.ev_join[1], D.spill_s));
    HIPC(hipStreamWaitEvent(D.comp, D.ev_join[0], 0));
    HIPC(hipStreamWaitEvent(D.comp, D.ev_join[1], 0));
    hipEvent_t a = nullptr, b = nullptr;
    if (timed) {
      a = D.timing_event();
      b = D.timing_event();
      HIPC(hipEventRecord(a, D.comp));
    }
    HIPC(launch_finish(kp, D.arena, (char*)D.results, D.comp));
    if (timed) {
      HIPC(hipEventRecord(b, D.comp));
      D.tpairs.push_back({-1, 0, 0, -1, 0.0, a, b});
    }
  }
  n_launch++;
  HIPC(hipEventRecord(D.t1, D.comp));
  // the compute stream follows every transfer and the results are on the host
  HIPC(hipStreamSynchronize(D.comp));
  float ms = 0;
  HIPC(hipEventElapsedTime(&ms, D.t0, D.t1));
  c.corr_host.assign((const double*)D.results, (const double*)D.results + kp.corr_bytes / 8);
  c.sums_host.assign((const double*)((const char*)D.results + kp.corr_bytes),
                     (const double*)((const char*)D.results + kp.corr_bytes) + kp.sums_bytes / 8);
  double t_hec = 0, t_kern = 0, t_copy = 0;
  if (timed) {
    c.records.clear();
    for (const Device::TPair& pr : D.tpairs) {
      float x = 0;
      HIPC(hipEventElapsedTime(&x, pr.a, pr.b));
      cdag_launch_record r{};
      r.step = pr.step;
      r.ms = x;
      if (pr.launch == -2) {
        r.type = pr.type;
        r.kinds = pr.kinds;
        r.n_items = 1;
        r.bytes = pr.bytes;
        c.records.push_back(r);
        t_copy += x * 1e-3;
        continue;
      }
      t_kern += x * 1e-3;
      const Launch& L = pr.launch >= 0 ? kp.launches[pr.launch] : kp.xsum;
      r.type = L.type;
      r.variant = L.type == L_HEC ? L.tile : 0;
      r.interior = L.type == L_HEC ? L.interior : 0;
      r.kinds = L.kinds;
      r.n_items = L.n_items;
      r.flops = L.flops;
      r.bytes = L.bytes;
      r.trace_items = L.tr_n_items;
      r.trace_flops = L.tr_flops;
      r.trace_bytes = L.tr_bytes;
      c.records.push_back(r);
      if (L.type == L_HEC) t_hec += x * 1e-3;
    }
  }
  int64_t n_hec = 0;
  for (const Launch& L : kp.launches) n_hec += L.type == L_HEC;
  st->t_hec_s = t_hec;
  st->t_kernels_s = t_kern;
  st->t_copy_s = t_copy;
  st->arena_highwater = kp.total_bytes;
  st->hec_flops = kp.hec_flops;
  st->hec_bytes = kp.hec_bytes;
  st->n_hec_launches = n_hec;
  st->t_total_s = now() - tw0;
  st->t_device_s = ms * 1e-3;
  st->n_launches = n_launch;
  st->n_graph_segments = n_segments;
}

// ---------------------------------------------------------------- no allocation
namespace {
// The one-stream walk with every byte in the static scratch: leaf uploads copy
// the library's interleaved host copy into a staging range at the end of the
// scratch and convert it into place on the device.
struct StaticOps {
  const Ctx& c;
  int prec;
  char* base;
  int64_t staging;    // offset of the staging range in the scratch
  hipStream_t st;

  void wait(int, int, int64_t, int64_t) {}
  void record(int, int64_t) {}
  void wait_pass(int, int, int64_t, int64_t) {}
  void record_pass(int, int64_t, int64_t) {}
  void upload_leaf(int64_t u, int64_t dev_off) const {
    const bool src_double = c.leaf_dtype[u] == CDAG_C128;
    const int64_t nt = c.dag.nt[u], e = c.dag.elems(u) / nt;
    HIPC(hipMemcpyAsync(base + staging, c.leaf_data[u].data(), c.leaf_data[u].size(), hipMemcpyHostToDevice, st));
    HIPC(launch_to_planar(src_double, prec == CDAG_FP64, base + staging, base + dev_off, nt, e, st));
  }
  void transfer(const PlanRec& r, const PassMap&, int64_t) {
    if (r.op != OP_H2D || !c.dag.is_leaf(r.node)) throw Error(CDAG_E_STATE, "static execute: a spill in the plan");
    upload_leaf(r.node, r.dev_off);
  }
  int64_t launch(int64_t g, const PassMap&) { return launch_step(c.kplan, g, prec, base, st, nullptr); }
};
}  // namespace

void device_execute_static(Ctx& c, int prec, cdag_exec_stats* st) {
  Device& D = *c.dev;
  const double tw0 = now();
  HIPC(hipSetDevice(D.device));
  char* base = scratch_address(D.device);
  if (!base) throw Error(CDAG_E_STATE, "static scratch not set up on this device");
  const Plan& p = c.plan;
  const KernelPlan& kp = c.kplan;
  if (p.chunks() != 1) throw Error(CDAG_E_STATE, "static execute runs whole tensors (t_chunks 1)");
  if (p.n_d2h > 0) throw Error(CDAG_E_BUDGET, "static execute: the plan spills to host memory");
  int64_t staging = 0;
  for (int64_t u = 0; u < c.dag.n_leaves; ++u) staging = std::max<int64_t>(staging, (int64_t)c.leaf_data[u].size());
  const int64_t stage_off = (kp.total_bytes + 255) / 256 * 256;
  if (stage_off + staging > kScratchBytes)
    throw Error(CDAG_E_NOMEM, "static execute needs " + std::to_string(stage_off + staging) +
                                  " bytes of device memory, the static scratch holds " + std::to_string(kScratchBytes));
  if ((int64_t)c.corr_host.size() * 8 < kp.corr_bytes || (int64_t)c.sums_host.size() * 8 < kp.sums_bytes)
    throw Error(CDAG_E_STATE, "static execute: result buffers not sized by the plan");
  hipStream_t s = D.comp;
  StaticOps ops{c, prec, base, stage_off, s};
  // descriptor tables (every call: another context may have used the scratch)
  HIPC(hipMemcpyAsync(base + kp.blob_off, kp.blob.data(), kp.blob.size(), hipMemcpyHostToDevice, s));
  if (c.leaves_resident)
    for (int64_t u = 0; u < c.dag.n_leaves; ++u) ops.upload_leaf(u, p.leaf_off[u]);
  const int64_t G = p.n_xsteps();
  int64_t n_launch = walk_steps(c, 0, G, true, false, ops);
  HIPC(launch_finish(kp, base, nullptr, s));
  ++n_launch;
  HIPC(hipMemcpyAsync(c.corr_host.data(), base + kp.corr_off, (size_t)kp.corr_bytes, hipMemcpyDeviceToHost, s));
  HIPC(hipMemcpyAsync(c.sums_host.data(), base + kp.sums_off, (size_t)kp.sums_bytes, hipMemcpyDeviceToHost, s));
  HIPC(hipStreamSynchronize(s));
  int64_t n_hec = 0;
  for (const Launch& L : kp.launches) n_hec += L.type == L_HEC;
  st->hec_flops = kp.hec_flops;
  st->hec_bytes = kp.hec_bytes;
  st->n_hec_launches = n_hec;
  st->n_launches = n_launch;
  st->arena_highwater = stage_off + staging;
  st->t_total_s = now() - tw0;
}

}  // namespace cdag
