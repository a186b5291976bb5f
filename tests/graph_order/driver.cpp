// Walks seeded plans in one to eight passes over the time slices with the graph
// form of the executor, its nodes recorded instead of added to a HIP graph, and
// checks the dependencies that GraphOrder gives them (tests/test_graph_order.py).
//   - Without copy nodes the graph is a plain sequence: each node depends on the
//     one before it and on nothing else, and there are as many nodes as launches.
//   - With transfers as copy nodes (all of them, or the large ones), any two
//     nodes that touch the same bytes, one of them writing, are ordered.
#include <cstdio>
#include <cstdlib>
#include <vector>

#ifndef ORDER_HEADER
#define ORDER_HEADER "runtime/graph_order.hpp"
#endif
#include ORDER_HEADER
#include "ctx.hpp"

using namespace cdag;

namespace {
uint64_t g_state = 0x9e3779b97f4a7c15ULL;
int pick(int n) {                           // splitmix64
  uint64_t z = (g_state += 0x9e3779b97f4a7c15ULL);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
  return (int)((z ^ (z >> 31)) % (uint64_t)n);
}

struct Access {
  int space;                                // arena, spill
  int64_t lo, hi;
  bool write;
};
struct NodeRec {
  std::vector<int> deps;
  std::vector<Access> acc;
};

// The graph form with node numbers: transfers of more than `copy_bytes` a step
// and direction are copy nodes, others one chain node; a step's kernels are two
// chain nodes, so that a node without accesses of its own is in the chain.
struct RecordOps {
  const Ctx& c;
  int64_t copy_bytes;
  GraphOrder<int> order;
  std::vector<NodeRec> nodes{};
  std::vector<NodeRec> moves[kStreams]{};
  int64_t bytes[kStreams] = {0, 0, 0}, launches = 0;

  RecordOps(const Ctx& ctx, int64_t limit)
      : c(ctx), copy_bytes(limit), order(ctx.plan.n_xsteps(), ctx.plan.chunks()) {}
  void add(int r, bool in_chain, NodeRec n) {
    order.deps_of(r, in_chain, &n.deps);
    nodes.push_back(std::move(n));
    order.added(r, in_chain, (int)nodes.size() - 1);
    ++launches;
  }
  void wait(int to, int from, int64_t g, int64_t) { order.wait(to, from, g); }
  void wait_pass(int to, int from, int64_t k, int64_t) { order.wait_pass(to, from, k); }
  void record_pass(int r, int64_t k, int64_t) { order.record_pass(r, k); }
  void record(int r, int64_t g) {
    if (!moves[r].empty() && bytes[r] <= copy_bytes) {
      NodeRec all;
      for (auto& m : moves[r]) all.acc.insert(all.acc.end(), m.acc.begin(), m.acc.end());
      add(r, true, all);
    } else {
      for (auto& m : moves[r]) add(r, false, m);
    }
    moves[r].clear();
    bytes[r] = 0;
    order.record(r, g);
  }
  void transfer(const PlanRec& r, const PassMap& m, int64_t) {
    const int s = r.op == OP_D2H ? S_D2H : S_H2D;
    const int64_t n = m.bytes(r.node), dev = m.dev(r.dev_off), host = m.host(r.host_off);
    NodeRec rec;
    rec.acc.push_back({0, dev, dev + n, s == S_H2D});
    if (!c.dag.is_leaf(r.node)) rec.acc.push_back({1, host, host + n, s == S_D2H});
    moves[s].push_back(rec);
    bytes[s] += n;
  }
  int64_t launch(int64_t g, const PassMap& m) {
    const Plan::Program& prog = c.plan.program(m.k);
    const int64_t s = g - c.plan.xfirst(m.k);
    NodeRec rec;
    for (int64_t i = prog.off[s]; i < prog.off[s + 1]; ++i) {
      const PlanRec& r = prog.recs[i];
      if (r.op != OP_EXEC) continue;
      const int64_t x[2] = {c.dag.left[r.node], c.dag.right[r.node]}, at[2] = {r.a_off, r.b_off};
      for (int j = 0; j < 2; ++j) {
        const int64_t lo = m.operand(x[j], at[j]);
        rec.acc.push_back({0, lo, lo + m.bytes(x[j]), false});
      }
      if (c.dag.kind[r.node] != HCA) rec.acc.push_back({0, m.dev(r.dev_off), m.dev(r.dev_off) + m.bytes(r.node), true});
    }
    add(S_COMP, true, NodeRec{});
    add(S_COMP, true, rec);
    return 2;
  }
};

void build_case(Ctx& c, int nm, int nb, int n_graphs, int n, int nt) {
  std::vector<LeafIn> leaves;
  for (int i = 0; i < nm; ++i) leaves.push_back({2, n, nt});
  for (int i = 0; i < nb; ++i) leaves.push_back({3, n, nt});
  std::vector<std::vector<OpIn>> ops(n_graphs);
  std::vector<GraphIn> graphs;
  for (int g = 0; g < n_graphs; ++g) {
    std::vector<OpIn>& o = ops[g];
    if (nb >= 2 && g % 2) {
      const int a = pick(nb), b = (a + 1 + pick(nb - 1)) % nb, x = pick(nm), y = (x + 1 + pick(nm - 1)) % nm;
      o = {{K32, nm + a, x}, {K33, -1, nm + b}, {HCA, -2, y}};
    } else {
      const int len = 4 + pick(3), first = pick(nm);
      int cur = first;
      for (int k = 1; k + 1 < len; ++k) {
        o.push_back({K22, cur, (first + k * (1 + g % 2)) % nm});
        cur = -(int)o.size();
      }
      o.push_back({HCA, cur, (first + (len - 1) * (1 + g % 2)) % nm});
    }
  }
  for (auto& o : ops) graphs.push_back({(int32_t)o.size(), 0, o.data(), 1.0, 0.0});
  c.dag = build(leaves, graphs);
  c.built = true;
  c.order = sched_tree(c.dag, 16, false);
  c.scheduled = true;
  c.leaf_dtype.assign(leaves.size(), CDAG_C128);
}

int64_t unordered_pairs(const std::vector<NodeRec>& nodes) {
  const size_t n = nodes.size(), words = (n + 63) / 64;
  std::vector<std::vector<uint64_t>> before(n, std::vector<uint64_t>(words, 0));
  for (size_t i = 0; i < n; ++i)
    for (int d : nodes[i].deps) {
      before[i][d / 64] |= 1ULL << (d % 64);
      for (size_t w = 0; w < words; ++w) before[i][w] |= before[d][w];
    }
  int64_t bad = 0;
  for (size_t i = 0; i < n; ++i)
    for (size_t j = 0; j < i; ++j) {
      if (before[i][j / 64] >> (j % 64) & 1) continue;
      for (const Access& a : nodes[i].acc)
        for (const Access& b : nodes[j].acc)
          if (a.space == b.space && a.lo < b.hi && b.lo < a.hi && (a.write || b.write)) ++bad;
    }
  return bad;
}
}  // namespace

int main() {
  int fails = 0, spilling = 0, mixed = 0;
  for (int baryons : {0, 4})
    for (int64_t chunks = 1; chunks <= 8; ++chunks)
      for (int64_t look : {(int64_t)0, (int64_t)16, INT64_MAX})
        for (int part : {0, 2, 3}) {        // unlimited memory, or 1 / part of the order's live peak per pass
          Ctx c;
          build_case(c, 6, baryons, 14, 8, 840);
          c.use_graphs = 2;
          c.t_chunks = chunks;
          c.wave_lookahead = look;
          const int64_t peak = memsim(c.dag, c.order, 16).peak_live;
          if (part > 0) c.budget = chunks > 1 ? 2 * (peak / chunks) / part : peak / part;
          try {
            ensure_plan(c, CDAG_FP64, 1);
          } catch (const Error& e) {
            if (e.code == CDAG_E_BUDGET) continue;
            throw;
          }
          spilling += c.plan.n_d2h > 0;
          const int64_t big = c.plan.tsize(c.dag, c.dag.n_leaves - 1);
          for (int64_t limit : {INT64_MAX, (int64_t)0, big}) {
            RecordOps ops(c, limit);
            walk_steps(c, 0, c.plan.n_xsteps(), false, false, ops);
            if (limit == INT64_MAX) {
              bool plain = !ops.order.copies() && (int64_t)ops.nodes.size() == ops.launches;
              for (size_t i = 0; i < ops.nodes.size(); ++i)
                plain &= i == 0 ? ops.nodes[i].deps.empty() : ops.nodes[i].deps == std::vector<int>{(int)i - 1};
              if (!plain) {
                std::printf("no plain sequence: baryons %d passes %ld lookahead %ld part %d\n", baryons, (long)chunks,
                            (long)look, part);
                ++fails;
              }
            } else {
              mixed += ops.order.copies();
              const int64_t bad = unordered_pairs(ops.nodes);
              if (bad > 0) {
                std::printf("%ld unordered accesses: baryons %d passes %ld lookahead %ld part %d limit %ld\n", (long)bad,
                            baryons, (long)chunks, (long)look, part, (long)limit);
                ++fails;
              }
            }
          }
        }
  if (fails == 0 && spilling > 10 && mixed > 50) std::printf("graph order driver: ok\n");
  else std::printf("fails %d, spilling plans %d, graphs with copies %d\n", fails, spilling, mixed);
  return fails != 0;
}
