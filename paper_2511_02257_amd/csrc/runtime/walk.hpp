// The order in which a placed plan is issued on three streams (kernels, uploads,
// spills), apart from what issues it: Ops makes HIP calls, graph nodes or trace
// records of it (executor.hip).  Pure host code.
#pragma once

#include <algorithm>
#include <cstdint>

#include "../ctx.hpp"

namespace cdag {

// Stream roles; trace records and event ids use these numbers.
enum StreamRole : int { S_COMP = 0, S_H2D = 1, S_D2H = 2, kStreams = 3 };

// Where pass k of a time-chunked execution keeps its data: the tensor pool and
// workspace of half k % 2 of the arena, half k % 2 of the host spill pool, and
// slices [k nt / C, (k + 1) nt / C) of every tensor (bytes(u) per pass).
struct PassMap {
  const Ctx& c;
  int64_t k, dev_shift, host_shift;
  PassMap(const Ctx& ctx, int64_t pass)
      : c(ctx), k(pass), dev_shift((pass % 2) * ctx.kplan.half_bytes),
        host_shift((pass % 2) * ctx.plan.host_spill_bytes) {}
  int64_t bytes(int64_t u) const { return c.plan.tsize(c.dag, u); }
  int64_t dev(int64_t off) const { return off + dev_shift; }
  int64_t host(int64_t off) const { return off + host_shift; }
  int64_t stage(int64_t u) const { return k * bytes(u); }   // in the leaf's staging buffer
  // arena offset of operand x planned at `planned`: a resident leaf's slices of
  // this pass, else the planned offset in the pass's half
  int64_t operand(int64_t x, int64_t planned) const {
    if (c.plan.opts.leaves_resident && c.dag.is_leaf(x)) return c.plan.leaf_off[x] + k * bytes(x);
    return dev(planned);
  }
};

// Walk global execution steps [g0, g1), step s of pass k's program at a time: each
// step's spills (after the kernels that last touched the tensor and any upload
// still reading the host range), its uploads (after the kernels and spills
// that last used the arena range, and the spill that wrote a re-uploaded
// tensor), then its kernels (after the step's uploads and any spill still
// reading an output's memory).  With one_stream (how one-stream segments are
// captured) every dependency is the stream order and no event is used.  In a
// captured segment, waits on steps before g0 are left out: the segments' graphs
// run one after another on one stream, so everything before g0 has finished
// when the segment starts.  Ops issues the work (HipOps) or records it
// (TraceOps).
template <class Ops>
int64_t walk_steps(const Ctx& c, int64_t g0, int64_t g1, bool one_stream, bool in_capture, Ops& ops) {
  const Plan& p = c.plan;
  const int64_t C = p.chunks();
  // waited[to][from]: newest step of stream `from` that stream `to` has waited
  // for; events of one stream complete in step order, so older ones are implied
  int64_t waited[kStreams][kStreams];
  for (auto& row : waited)
    for (auto& x : row) x = in_capture ? g0 - 1 : -1;
  auto wait = [&](int to, int from, int64_t g) {
    if (one_stream || g < 0 || g <= waited[to][from]) return;
    ops.wait(to, from, g, g);
    waited[to][from] = g;
  };
  int64_t n_launch = 0;
  for (int64_t g = g0; g < g1; ++g) {
    const int64_t k = p.pass_of(g), kS = p.xfirst(k), s = g - kS;
    const Plan::Program& prog = p.program(k);
    const PassMap m(c, k);
    auto at = [&](int64_t step) { return step >= 0 ? kS + step : -1; };
    if (s == 0 && k >= 2 && !one_stream && !(in_capture && p.xfirst(k - 1) <= g0)) {
      // pass k - 2 used the same half of the arena and of the spill pool
      ops.wait_pass(S_H2D, S_COMP, k - 2, g);
      ops.wait_pass(S_H2D, S_D2H, k - 2, g);
      ops.wait_pass(S_D2H, S_H2D, k - 2, g);
      ops.wait_pass(S_COMP, S_D2H, k - 2, g);
    }
    bool any_d2h = false, any_h2d = false;
    int64_t alloc_d2h = -1;
    for (int64_t ri = prog.off[s]; ri < prog.off[s + 1]; ++ri) {
      const PlanRec& r = prog.recs[ri];
      if (r.op != OP_D2H) continue;
      wait(S_D2H, S_COMP, at(r.wait_comp));
      wait(S_D2H, S_H2D, at(r.wait_h2d));
      ops.transfer(r, m, g);
      any_d2h = true;
    }
    if (any_d2h && !one_stream) ops.record(S_D2H, g);
    for (int64_t ri = prog.off[s]; ri < prog.off[s + 1]; ++ri) {
      const PlanRec& r = prog.recs[ri];
      if (r.op == OP_H2D) {
        wait(S_H2D, S_COMP, at(r.wait_comp));
        wait(S_H2D, S_D2H, at(r.wait_d2h));
        ops.transfer(r, m, g);
        any_h2d = true;
      } else if (r.op == OP_ALLOC) {
        alloc_d2h = std::max(alloc_d2h, at(r.wait_d2h));
      }
    }
    if (any_h2d && !one_stream) ops.record(S_H2D, g);
    if (any_h2d) wait(S_COMP, S_H2D, g);
    wait(S_COMP, S_D2H, alloc_d2h);
    n_launch += ops.launch(g, m);
    if (!one_stream) {
      ops.record(S_COMP, g);
      if (s == prog.n() - 1 && k + 2 < C)
        for (int r = 0; r < kStreams; ++r) ops.record_pass(r, k, g);
    }
  }
  return n_launch;
}

}  // namespace cdag
