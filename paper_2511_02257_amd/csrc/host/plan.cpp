// Budgeted execution plan: wave cut, next-use eviction, uploads and releases,
// then physical placement of every allocation in the device arena.
//
// The paper counts evictions, transfers and transfer bytes (Sec. IV-C) but its
// memory manager is not specified; this plan is the engine's own policy:
//   steps     one per contraction, or waves of ready contractions in schedule
//             order (cut_waves); with lookahead 0 the order is kept and a wave
//             closes before c when (a) an operand of c is produced in the wave,
//             (b) the bytes of the wave's distinct operands and outputs with c
//             would exceed the budget, or (c) the wave holds wave_max;
//   eviction  while used + need > budget, evict the resident tensor that is
//             not an operand of the step with the furthest next use (ties:
//             larger size, then smaller id); leaves and already-spilled
//             intermediates are dropped, other intermediates copied to the
//             host once;
//   then      upload missing operands (ascending id), allocate outputs (a
//             root's output is 0 bytes), run, free what nothing later needs.
#include <algorithm>
#include <map>
#include <set>
#include <tuple>

#include "host.hpp"
#include "../../../include/cdag.h"

namespace cdag {

std::vector<std::vector<int64_t>> cut_waves(const Dag& d, const std::vector<int64_t>& order,
                                            const std::vector<int64_t>& size, int64_t budget,
                                            int64_t wave_max, int64_t lookahead) {
  // A contraction is ready when both operands are leaves or outputs of earlier
  // waves.  Scanning unplaced contractions in schedule order, a wave takes each
  // ready one and passes over at most `lookahead` not-ready ones; it closes at
  // the next not-ready one, when the distinct operand and output bytes would
  // exceed the budget, or at wave_max contractions.
  std::vector<std::vector<int64_t>> waves;
  const int64_t n = (int64_t)order.size();
  std::vector<char> placed(n, 0), produced(d.n_nodes(), 0);
  std::vector<int64_t> member(d.n_nodes(), -1);
  int64_t start = 0, wid = 0;
  auto ready = [&](int64_t x) { return d.is_leaf(x) || produced[x]; };
  while (start < n) {
    std::vector<int64_t> wave;
    int64_t bytes = 0, skipped = 0;
    for (int64_t pos = start; pos < n; ++pos) {
      if (placed[pos]) continue;
      const int64_t c = order[pos], l = d.left[c], r = d.right[c];
      if (!ready(l) || !ready(r)) {
        if (++skipped > lookahead) break;
        continue;
      }
      int64_t extra = 0;
      for (int64_t x : {l, r, c})
        if (member[x] != wid) extra += size[x];
      if (!wave.empty() && (bytes + extra > budget || (int64_t)wave.size() >= wave_max)) break;
      for (int64_t x : {l, r, c}) member[x] = wid;
      bytes += extra;
      wave.push_back(c);
      placed[pos] = 1;
    }
    for (int64_t c : wave) produced[c] = 1;
    waves.push_back(std::move(wave));
    ++wid;
    while (start < n && placed[start]) ++start;
  }
  return waves;
}

PlanTotals plan_totals(const Plan& p) {
  const int64_t C = p.chunks();
  return {C * (int64_t)p.steps.size(), p.halves() * p.peak_resident, C * p.n_evict, C * p.n_h2d,
          C * p.h2d_bytes, C * p.n_d2h, C * p.d2h_bytes};
}

Plan make_plan(const Dag& d, const std::vector<int64_t>& order, const PlanOpts& o) {
  const int64_t n = d.n_nodes();
  if (o.t_chunks < 1) throw Error(CDAG_E_INVALID, "t_chunks must be >= 1");
  for (int64_t u = 0; u < n && o.t_chunks > 1; ++u)
    if (d.nt[u] % o.t_chunks != 0)
      throw Error(CDAG_E_INVALID, "t_chunks must divide the number of time slices of every tensor");
  Plan p;
  p.opts = o;
  // one pass: tensors of nt / t_chunks slices in one half of the budget
  const int64_t budget = o.t_chunks > 1 ? o.budget / 2 : o.budget;
  std::vector<int64_t> size(n);
  for (int64_t u = 0; u < n; ++u) size[u] = p.tsize(d, u);
  if (o.leaves_resident)
    for (int64_t u = 0; u < d.n_leaves; ++u) size[u] = 0;
  if (o.batched) {
    p.steps = cut_waves(d, order, size, budget, o.wave_max, o.lookahead);
  } else {
    p.steps.reserve(order.size());
    for (int64_t c : order) p.steps.push_back({c});
  }
  const int64_t S = (int64_t)p.steps.size();
  // uses[x]: ascending distinct steps where x is an operand
  std::vector<int64_t> cnt(n + 1, 0), last(n, -1);
  for (int64_t s = 0; s < S; ++s)
    for (int64_t c : p.steps[s])
      for (int64_t x : {d.left[c], d.right[c]})
        if (last[x] != s) { last[x] = s; cnt[x]++; }
  std::vector<int64_t> use_off(n + 1, 0);
  for (int64_t u = 0; u < n; ++u) use_off[u + 1] = use_off[u] + cnt[u];
  std::vector<int64_t> uses(use_off[n]), fill(use_off.begin(), use_off.end() - 1);
  std::fill(last.begin(), last.end(), -1);
  for (int64_t s = 0; s < S; ++s)
    for (int64_t c : p.steps[s])
      for (int64_t x : {d.left[c], d.right[c]})
        if (last[x] != s) { last[x] = s; uses[fill[x]++] = s; }
  std::vector<int64_t> ptr(use_off.begin(), use_off.end() - 1);
  auto next_use_after = [&](int64_t x, int64_t s) -> int64_t {
    while (ptr[x] < use_off[x + 1] && uses[ptr[x]] <= s) ++ptr[x];
    return ptr[x] < use_off[x + 1] ? uses[ptr[x]] : INT64_MAX;
  };

  std::vector<int64_t> remaining(n);
  for (int64_t u = 0; u < n; ++u) remaining[u] = d.n_parents(u);
  std::vector<char> resident(n, 0), host_copy(n, 0), pinned(n, 0);
  // evictable residents keyed (next use, size, -id); the max is the victim
  using Key = std::tuple<int64_t, int64_t, int64_t>;
  std::set<Key> cand;
  std::vector<int64_t> key_nu(n, -1);
  auto cand_insert = [&](int64_t x, int64_t nu) { key_nu[x] = nu; cand.insert({nu, size[x], -x}); };
  auto cand_erase = [&](int64_t x) { cand.erase({key_nu[x], size[x], -x}); };
  if (o.leaves_resident)
    for (int64_t u = 0; u < d.n_leaves; ++u) resident[u] = 1;   // never candidates

  int64_t used = 0;
  std::vector<int64_t> operands;
  p.rec_off.reserve(S + 1);
  for (int64_t s = 0; s < S; ++s) {
    p.rec_off.push_back((int64_t)p.recs.size());
    const auto& wave = p.steps[s];
    operands.clear();
    for (int64_t c : wave) { operands.push_back(d.left[c]); operands.push_back(d.right[c]); }
    std::sort(operands.begin(), operands.end());
    operands.erase(std::unique(operands.begin(), operands.end()), operands.end());
    int64_t need = 0;
    for (int64_t x : operands) {
      pinned[x] = 1;
      if (!resident[x]) need += size[x];
    }
    for (int64_t c : wave) need += size[c];
    // pinned residents are keyed by next use == s, below every other candidate
    for (int64_t x : operands)
      if (resident[x] && !(o.leaves_resident && d.is_leaf(x))) { cand_erase(x); cand_insert(x, s); }
    while (used + need > budget) {
      if (cand.empty()) throw Error(CDAG_E_BUDGET, "step " + std::to_string(s) + " does not fit in the budget");
      auto it = std::prev(cand.end());
      int64_t v = -std::get<2>(*it);
      if (pinned[v]) throw Error(CDAG_E_BUDGET, "step " + std::to_string(s) + " does not fit in the budget");
      cand.erase(it);
      if (d.is_leaf(v) || host_copy[v]) {
        p.recs.push_back({OP_DROP, v, s});
      } else {
        p.recs.push_back({OP_D2H, v, s});
        p.n_d2h++;
        p.d2h_bytes += size[v];
        host_copy[v] = 1;
      }
      p.n_evict++;
      resident[v] = 0;
      used -= size[v];
    }
    for (int64_t x : operands) {
      if (resident[x]) continue;
      if (!d.is_leaf(x) && !host_copy[x]) throw Error(CDAG_E_STATE, "plan: intermediate lost");
      p.recs.push_back({OP_H2D, x, s});
      p.n_h2d++;
      p.h2d_bytes += size[x];
      resident[x] = 1;
      used += size[x];
      cand_insert(x, s);
    }
    for (int64_t c : wave) {
      if (d.kind[c] == HCA) continue;
      p.recs.push_back({OP_ALLOC, c, s});
      resident[c] = 1;
      used += size[c];
    }
    p.peak_resident = std::max(p.peak_resident, used);
    for (int64_t c : wave) p.recs.push_back({OP_EXEC, c, s});
    for (int64_t c : wave) { remaining[d.left[c]]--; remaining[d.right[c]]--; }
    for (int64_t x : operands) {
      pinned[x] = 0;
      if (o.leaves_resident && d.is_leaf(x)) continue;
      cand_erase(x);
      if (remaining[x] == 0) {
        p.recs.push_back({OP_FREE, x, s});
        resident[x] = 0;
        host_copy[x] = 0;
        used -= size[x];
      } else {
        cand_insert(x, next_use_after(x, s));
      }
    }
    for (int64_t c : wave)
      if (d.kind[c] != HCA) cand_insert(c, next_use_after(c, s));
  }
  p.rec_off.push_back((int64_t)p.recs.size());
  return p;
}

// ---------------------------------------------------------------- placement
namespace {
constexpr int64_t kAlign = 256;
int64_t align_up(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Best-fit allocator over [0, inf) that remembers, per free range, the last
// compute step that touched the memory and the last transfer that read it
// (device ranges: a spill; host ranges: an upload).  Below `cap` bytes it takes
// fresh memory first, and then the large enough block whose last use is oldest
// (of equally old ones the smallest).
class Pool {
 public:
  explicit Pool(int64_t cap = 0) : cap_(cap) {}
  struct Free { int64_t size, comp, copy; };
  int64_t top = 0;

  // Returns offset; *comp / *copy receive the waits inherited from the block.
  int64_t alloc(int64_t bytes, int64_t* comp, int64_t* copy) {
    bytes = align_up(std::max<int64_t>(bytes, 1));
    const bool fresh = cap_ > 0 && top + bytes <= cap_;
    int64_t off = -1;
    if (cap_ == 0) {
      const auto it = by_size_.lower_bound({bytes, -1});
      if (it != by_size_.end()) off = it->second;
    } else if (!fresh && !by_size_.empty() && by_size_.rbegin()->first >= bytes) {
      auto it = by_age_.begin();
      while (std::get<1>(*it) < bytes) ++it;
      off = std::get<2>(*it);
    }
    if (off >= 0) {
      const Free f = take(off);
      if (f.size > bytes) put(off + bytes, {f.size - bytes, f.comp, f.copy});
      *comp = f.comp;
      *copy = f.copy;
      return off;
    }
    // extend from a free block that ends at the top, else from fresh memory
    if (!free_.empty() && !fresh) {
      const auto last = std::prev(free_.end());
      if (last->first + last->second.size == top) {
        off = last->first;
        const Free f = take(off);
        top = off + bytes;
        *comp = f.comp;
        *copy = f.copy;
        return off;
      }
    }
    off = top;
    top += bytes;
    *comp = -1;
    *copy = -1;
    return off;
  }
  void release(int64_t off, int64_t bytes, int64_t comp, int64_t copy) {
    Free f{align_up(std::max<int64_t>(bytes, 1)), comp, copy};
    const auto nx = free_.lower_bound(off);
    if (nx != free_.end() && off + f.size == nx->first) join(&f, take(nx->first));   // merge right
    const auto at = free_.lower_bound(off);
    if (at != free_.begin()) {                                                      // merge left
      const auto pv = std::prev(at);
      if (pv->first + pv->second.size == off) {
        off = pv->first;
        join(&f, take(off));
      }
    }
    put(off, f);
  }

 private:
  int64_t cap_;
  std::map<int64_t, Free> free_;                             // offset -> block
  std::set<std::pair<int64_t, int64_t>> by_size_;            // (size, offset)
  std::set<std::tuple<int64_t, int64_t, int64_t>> by_age_;   // (comp, size, offset); with a cap only

  void put(int64_t off, const Free& f) {
    free_[off] = f;
    by_size_.insert({f.size, off});
    if (cap_ > 0) by_age_.insert({f.comp, f.size, off});
  }
  Free take(int64_t off) {
    const auto it = free_.find(off);
    const Free f = it->second;
    free_.erase(it);
    by_size_.erase({f.size, off});
    if (cap_ > 0) by_age_.erase({f.comp, f.size, off});
    return f;
  }
  static void join(Free* f, const Free& o) {
    f->size += o.size;
    f->comp = std::max(f->comp, o.comp);
    f->copy = std::max(f->copy, o.copy);
  }
};
}  // namespace

namespace {
// Pool up to which placement takes fresh memory to keep contractions of
// different plan steps from waiting for one another's, and the most that it
// takes beyond the tightest pool: half of the 256 MB last-level cache, so that
// intermediates still meet there.
constexpr int64_t kSpreadBytes = 128LL << 20;
// Uploads of one execution step in overlapping issue: at least this, and a
// quarter of what the plan step uploads.
constexpr int64_t kStageBytes = 32LL << 20;
// A plan of more than kFewSteps steps of kLongStep seconds of contractions on
// average is issued step by step (see place()).
constexpr int64_t kFewSteps = 32;
constexpr double kLongStep = 100e-6;

// modelled_time(): launch and latency of a step, compute units.
constexpr double kStepTime = 7e-6, kUnits = 256;
// Shares of a modelled time that another cut has to stay below to be taken in its
// place: any cut for the plan steps' (or, where contractions fill kFilled of it,
// so that a cut costs little), plan steps for STAGED in the later passes, MERGED
// for either (see place()).
constexpr double kWorthCutting = 0.99, kFilled = 0.95, kBelowFilled = 0.998, kBelowStaged = 0.998, kBelowUncut = 0.98;

// How execution steps are cut (place()).
enum Cut { PLAN_STEPS, STAGED, MERGED };

// One placement of the pool, with at most `cap` bytes of it taken before memory
// is reused (0: tightest; the offsets then do not depend on the cut), and its
// program.  *staged (may be nullptr): whether a step's uploads are staged.
Plan::Program place_pool(const Dag& d, Plan& p, int64_t base, int64_t cap, Cut cut, bool* staged = nullptr) {
  const int64_t n = d.n_nodes();
  const bool merge = cut != PLAN_STEPS;
  Pool dev(cap), host;
  // last_touch: execution step of the last kernels that read or wrote the
  // tensor; spilled: that of the spill that wrote its host copy; uploaded: that
  // of the last upload that read that host copy; avail: first one whose kernels
  // may read it; out_after: first one whose kernels may write it
  std::vector<int64_t> off(n, -1), hoff(n, -1), last_touch(n, -1), spilled(n, -1), uploaded(n, -1);
  std::vector<int64_t> avail(n, 0), out_after(n, 0);
  // contractions in each execution step; room[k]: k while it has room for
  // another (wave_max), else a step on the way to the next that has
  std::vector<int64_t> in_step, room;
  auto with_room = [&](int64_t at) {
    for (;; at = room[at]) {
      for (int64_t k = (int64_t)room.size(); k <= at + 1; ++k) {
        in_step.push_back(0);
        room.push_back(k);
      }
      if (room[at] == at) return at;
      room[at] = room[room[at]];
    }
  };
  if (p.opts.leaves_resident)
    for (int64_t u = 0; u < d.n_leaves; ++u) off[u] = p.leaf_off[u];
  // A step with more uploads than one stage stages its smaller tensors first (a
  // contraction's small operand then does not hold it back): stage of each of
  // its uploads, -1 for the uploads of other steps.
  const int64_t R = (int64_t)p.recs.size();
  std::vector<int64_t> stage(p.steps.size(), INT64_MAX), stage_of(R, -1);
  for (size_t s = 0; merge && p.opts.overlap && s < p.steps.size(); ++s) {
    std::vector<int64_t> ups;
    int64_t bytes = 0, in_stage = 0, k = 0;
    for (int64_t i = p.rec_off[s]; i < p.rec_off[s + 1]; ++i)
      if (p.recs[i].op == OP_H2D) {
        bytes += p.tsize(d, p.recs[i].node);
        ups.push_back(i);
      }
    stage[s] = std::max<int64_t>(kStageBytes, bytes / 4);
    if (bytes <= stage[s]) continue;
    if (staged) *staged = true;
    std::stable_sort(ups.begin(), ups.end(), [&](int64_t a, int64_t b) {
      return p.tsize(d, p.recs[a].node) < p.tsize(d, p.recs[b].node);
    });
    for (int64_t i : ups) {
      const int64_t sz = p.tsize(d, p.recs[i].node);
      if (in_stage > 0 && in_stage + sz > stage[s]) {
        ++k;
        in_stage = 0;
      }
      in_stage += sz;
      stage_of[i] = k;
    }
  }
  int64_t up_x = 0, up_bytes = 0, last_x = -1;
  int64_t floor_x = 0, cur = -1, base_x = 0;   // STAGED: first execution step of plan step `cur`; its first upload's
  for (int64_t i = 0; i < R; ++i) {
    PlanRec& r = p.recs[i];
    const int64_t x = r.node, s = r.step, sz = p.tsize(d, x);
    if (s != cur) {
      cur = s;
      if (cut == STAGED) floor_x = last_x + 1;
      base_x = std::max(up_x, floor_x);
    }
    r.xstep = s;
    switch (r.op) {
      case OP_D2H: {
        int64_t c0, up;
        hoff[x] = host.alloc(sz, &c0, &up);
        r.host_off = hoff[x];
        r.dev_off = off[x];
        r.wait_comp = last_touch[x];
        r.wait_h2d = up;             // an upload still reading this host range
        dev.release(off[x] - base, sz, last_touch[x], s);
        spilled[x] = s;
        off[x] = -1;
        break;
      }
      case OP_DROP:
        r.dev_off = off[x];
        dev.release(off[x] - base, sz, last_touch[x], -1);
        off[x] = -1;
        break;
      case OP_H2D: {
        int64_t comp, spill;
        off[x] = base + dev.alloc(sz, &comp, &spill);
        r.dev_off = off[x];
        r.wait_comp = comp;          // kernels that last touched this memory
        if (d.is_leaf(x)) {
          r.host_off = -1;
          r.wait_d2h = spill;        // a spill still reading this memory
        } else {
          r.host_off = hoff[x];
          r.wait_d2h = std::max(spill, spilled[x]);   // ... and the spill that wrote the host copy
          uploaded[x] = s;
        }
        if (merge) {
          int64_t at = std::max({up_x, floor_x, comp + 1});
          if (stage_of[i] >= 0) at = std::max(base_x + stage_of[i], comp + 1);
          else if (at == up_x && up_bytes > 0 && up_bytes > stage[s] - sz) ++at;
          if (at > up_x) {
            up_bytes = 0;
            up_x = at;
          }
          up_bytes += sz;
          r.xstep = avail[x] = at;
        }
        break;
      }
      case OP_ALLOC: {
        int64_t comp, spill;
        off[x] = base + dev.alloc(sz, &comp, &spill);
        r.dev_off = off[x];
        r.wait_d2h = spill;          // a spill that last read this memory
        out_after[x] = comp + 1;     // kernels that last touched this memory
        break;
      }
      case OP_EXEC: {
        const int64_t a = d.left[x], b = d.right[x];
        r.a_off = off[a];
        r.b_off = off[b];
        r.dev_off = d.kind[x] == HCA ? -1 : off[x];
        if (merge) {
          const int64_t at = with_room(std::max({avail[a], avail[b], out_after[x], floor_x}));
          if (++in_step[at] >= p.opts.wave_max) room[at] = at + 1;
          r.xstep = at;
          avail[x] = at + 1;
        }
        for (int64_t u : {a, b, x}) last_touch[u] = std::max(last_touch[u], r.xstep);
        break;
      }
      case OP_FREE:
        dev.release(off[x] - base, sz, merge ? last_touch[x] : s, -1);
        off[x] = -1;
        if (hoff[x] >= 0) {
          host.release(hoff[x], sz, -1, uploaded[x]);
          hoff[x] = -1;
          uploaded[x] = -1;
        }
        break;
    }
    if (r.op == OP_EXEC || r.op == OP_H2D || r.op == OP_D2H) last_x = std::max(last_x, r.xstep);
  }
  p.pool_bytes = dev.top;
  p.host_spill_bytes = host.top;

  // An ALLOC has no work of its own; it goes with its contraction, whose
  // kernels wait for what it waits for.
  std::vector<int64_t> exec_x(n, -1);
  for (const PlanRec& r : p.recs)
    if (r.op == OP_EXEC) exec_x[r.node] = r.xstep;
  if (merge)
    for (PlanRec& r : p.recs)
      if (r.op == OP_ALLOC) r.xstep = exec_x[r.node];
  const int64_t X = merge ? last_x + 1 : (int64_t)p.steps.size();
  Plan::Program g;
  g.off.assign(X + 1, 0);
  auto issued = [](const PlanRec& r) { return r.op != OP_DROP && r.op != OP_FREE; };
  for (const PlanRec& r : p.recs)
    if (issued(r)) ++g.off[r.xstep + 1];
  for (int64_t k = 0; k < X; ++k) g.off[k + 1] += g.off[k];
  g.recs.resize(g.off[X]);
  std::vector<int64_t> at(g.off.begin(), g.off.end() - 1);
  for (bool transfers : {true, false})
    for (const PlanRec& r : p.recs)
      if (issued(r) && (r.op == OP_D2H || r.op == OP_H2D) == transfers) g.recs[at[r.xstep]++] = r;
  return g;
}

// Modelled time of the passes in eager issue: uploads one after another at the
// link's rate beside the kernels, each after the kernels that last used its
// memory (a pass after the one two before it), and each step's kernels after its
// uploads, for as long as its contractions take on the whole chip, or as its
// longest work item takes on one compute unit, whichever is more.  It is for
// putting cuts of one plan in order, not for their absolute times.
double modelled_time(const Dag& d, const Plan& p, const Plan::Program& first, const Plan::Program& later) {
  double up = 0, comp = 0, pass_end[2] = {0, 0};
  std::vector<double> done;                  // end of each step's kernels in the pass
  for (int64_t k = 0; k < p.chunks(); ++k) {
    const Plan::Program& g = k == 0 ? first : later;
    done.assign(g.n(), 0.0);
    up = std::max(up, pass_end[k % 2]);
    for (int64_t s = 0; s < g.n(); ++s) {
      double work = 0, item = 0, ready = comp;
      for (int64_t i = g.off[s]; i < g.off[s + 1]; ++i) {
        const PlanRec& r = g.recs[i];
        if (r.op == OP_H2D) {
          if (r.wait_comp >= 0) up = std::max(up, done[r.wait_comp]);
          up += (double)p.tsize(d, r.node) / p.opts.link_rate;
          ready = std::max(ready, up);
        } else if (r.op == OP_EXEC) {
          work += d.flops(r.node);
          if (!p.opts.item_flops.empty()) item = std::max(item, p.opts.item_flops[r.node]);
        }
      }
      done[s] = comp = ready + kStepTime + std::max(work / (double)p.chunks(), item * kUnits) / p.opts.flop_rate;
    }
    pass_end[k % 2] = comp;
  }
  return comp;
}
}  // namespace

// Execution steps.  A plan that runs in waves and never evicts need not be
// issued plan step by plan step (the plan's steps, counters and resident peak do
// not change):
//   MERGED  by data and memory dependencies: a contraction joins the first
//     execution step that is after its operands' kernels, its leaves' uploads
//     and the kernels that last touched the memory of its output; an upload goes
//     as early as its memory is free, in the plan's order.  Taken where that
//     makes fewer steps.  With lookahead 0 a wave ends at the first contraction
//     that needs one of its outputs, so a plan has hundreds of steps of a few
//     contractions each, at about 7 us of launch and latency a step, where the
//     dependencies are a few levels deep (46 graphs over any index pairs at N =
//     9: 72 plan steps, 4 execution steps, a pass 733 -> 96 us; 710 rank-4
//     graphs at N = 16 in two passes: 554 -> 30 steps, 17.2 -> 5.5 ms).
//   STAGED  a plan step with large uploads that run beside kernels in several
//     execution steps, each with a stage of the uploads and the contractions
//     whose operands are there by then, so that kernels start before the last
//     leaf.
// Where uploads are staged and MERGED does not make fewer steps, every cut adds
// steps, so it has to hide more of the uploads than they cost: a step takes at
// least as long as its longest work item (a K33 item with the whole K: 0.5 ms).
// The passes are modelled (modelled_time()), the first MERGED, which also moves
// later plan steps' contractions up between the stages, and the later ones
// STAGED, as the plan's steps or MERGED; the plan's steps stay unless a cut is
// modelled at least 1 % shorter (node order, the third line below: modelled 0.6 %
// shorter, measured 1.5 % longer), or 0.2 % where contractions fill the time
// (20,301 contractions in 16 passes: modelled 0.7 % shorter, 832 -> 818 ms).
// Where cuts are modelled alike the smaller launches of STAGED come out ahead by
// up to 1 % (the same in 8 passes 787 against 793 ms with the model 0.02 % the
// other way), and MERGED behind by up to 6 % (40.4 against 38.0, modelled 0.5 %
// the other way): hence the margins.  Measured (ms; baryon chains at N = 64, 8
// passes, FP64, K33 in whole items; by plan steps, then with the later passes as
// planned, STAGED, MERGED; * what is taken):
//   every ready contraction in a wave, 24 plan steps   38.0   36.7  36.0*  44.1
//   lookahead 64, 184                                  82.6*  82.7  86.1   92.5
//   node order, lookahead 16, 552                     258.8* 259.6 264.7  262.8
//   Sibling, lookahead 16, 576                        253.6* 253.8 266.3  266.6
// and five N families in 4 passes, lookahead 64: FP32   35.0   33.1  31.5   30.2*
//                                                FP64   65.2   66.0  62.4*  67.8
// Plans of many long steps keep their plan steps: launches cost them nothing,
// and a contraction that moves up leaves its output waiting for its consumer
// long enough to drop out of the last-level cache (20,301 contractions in 1,151
// waves of 0.75 ms, complex FP32: 0.87 s by plan steps, 0.95 MERGED; split BF16
// 0.61 and 0.68).
void place(const Dag& d, Plan& p) {
  p.leaf_off.assign(d.n_leaves, -1);
  int64_t base = 0;
  if (p.opts.leaves_resident) {
    // whole leaves: every pass reads its own slices of them
    for (int64_t u = 0; u < d.n_leaves; ++u) {
      p.leaf_off[u] = base;
      base += align_up(d.size(u, p.opts.elem_bytes));
    }
  }
  p.leaf_region_bytes = base;
  p.first = place_pool(d, p, base, 0, PLAN_STEPS);
  p.tight_pool_bytes = p.pool_bytes;
  double flops = 0;
  for (int64_t u = d.n_leaves; u < d.n_nodes(); ++u) flops += d.flops(u);
  const double t_pass = flops / (double)p.chunks() / p.opts.flop_rate;
  const bool many_long = p.first.n() > kFewSteps && t_pass > kLongStep * (double)p.first.n();
  if (p.opts.batched && p.n_evict == 0 && !many_long) {
    // merged where that makes fewer steps, in the tightest pool or else (without
    // a budget) in a wider one
    bool staged = false;
    Plan::Program merged = place_pool(d, p, base, 0, MERGED, &staged);
    if (p.opts.spread && p.opts.budget == INT64_MAX && p.pool_bytes < kSpreadBytes && merged.n() > 1) {
      Plan::Program wider = place_pool(d, p, base, kSpreadBytes, MERGED);
      // (past the cap, where it leaves no block large enough, it may still grow)
      const bool within = p.pool_bytes <= p.tight_pool_bytes + kSpreadBytes;
      if (within && wider.n() < std::min(merged.n(), p.first.n())) merged = std::move(wider);
      else place_pool(d, p, base, 0, PLAN_STEPS);   // back to the tightest placement
    }
    if (merged.n() < p.first.n()) {
      p.first = std::move(merged);
    } else if (staged) {
      const Plan::Program cut = place_pool(d, p, base, 0, STAGED);
      const Plan::Program* later = nullptr;
      const double t_plan = modelled_time(d, p, p.first, p.first);
      double best = t_plan * (t_pass * (double)p.chunks() > kFilled * t_plan ? kBelowFilled : kWorthCutting);
      const struct { const Plan::Program* cut; double below; } later_cuts[] = {
          {&cut, 1.0}, {&p.first, kBelowStaged}, {&merged, kBelowUncut}};
      for (const auto& l : later_cuts) {
        const double t = modelled_time(d, p, merged, *l.cut);
        if (t < best * (later != nullptr ? l.below : 1.0)) {
          best = t;
          later = l.cut;
        }
      }
      if (later != nullptr) {
        p.later = *later;
        p.first = std::move(merged);
        return;
      }
    }
  }
  p.later = p.first;
}

}  // namespace cdag
