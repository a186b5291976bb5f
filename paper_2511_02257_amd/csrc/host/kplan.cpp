// Launch planning (see kplan.hpp).
#include "kplan.hpp"

#include <algorithm>
#include <climits>
#include <cstring>

#include "../../../include/cdag.h"

namespace cdag {

namespace {
int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

template <class T>
int64_t put(std::vector<uint8_t>& blob, const T& v) {
  int64_t off = (int64_t)blob.size();
  blob.resize(blob.size() + sizeof(T));
  std::memcpy(blob.data() + off, &v, sizeof(T));
  return off;
}
}  // namespace

int64_t elem_bytes_of(int prec) { return prec == CDAG_FP64 ? 16 : 8; }

IndexMap index_map(const Spec& s, int n) {
  IndexMap m{};
  const int rl = s.rank_l, rr = s.rank_r, c = s.n_pairs, ro = rl + rr - 2 * c;
  auto stride = [&](int rank, int axis) {
    int64_t x = 1;
    for (int i = axis + 1; i < rank; ++i) x *= n;
    return x;
  };
  m.n = n;
  m.dk = c;
  int dm = 0, dn = 0;
  for (int a = 0; a < rl; ++a) {
    bool paired = false;
    for (int k = 0; k < c; ++k) paired |= s.pair_l[k] == a;
    if (!paired) m.a_m[dm++] = stride(rl, a);
  }
  for (int b = 0; b < rr; ++b) {
    bool paired = false;
    for (int k = 0; k < c; ++k) paired |= s.pair_r[k] == b;
    if (!paired) m.b_n[dn++] = stride(rr, b);
  }
  for (int k = 0; k < c; ++k) {
    m.a_k[k] = stride(rl, s.pair_l[k]);
    m.b_k[k] = stride(rr, s.pair_r[k]);
  }
  m.dm = dm;
  m.dn = dn;
  // natural output position q (m digits, then n digits) sits at output axis j
  // with perm[j] = q
  int64_t at[8];
  for (int j = 0; j < ro; ++j) at[s.perm[j]] = stride(ro, j);
  for (int d = 0; d < dm; ++d) m.c_m[d] = at[d];
  for (int d = 0; d < dn; ++d) m.c_n[d] = at[dm + d];
  // The order of an index's digits is free (it only renumbers the GEMM's rows
  // or columns): the output's unit-stride axis goes last in its index, so that a
  // tile covers runs of it.  Where the operand's own unit-stride axis is
  // another digit of that index, the larger of the two tensors decides (K
  // elements of the operand against `other` of the output per row or column).
  auto last_unit = [&](int nd, int64_t* oper, int64_t* out, int other) {
    int to = -1, oo = -1;
    for (int d = 0; d < nd; ++d) {
      if (out[d] == 1) to = d;
      if (oper[d] == 1) oo = d;
    }
    if (to < 0 || (oo >= 0 && oo != to && other < c)) return;
    std::swap(oper[to], oper[nd - 1]);
    std::swap(out[to], out[nd - 1]);
  };
  last_unit(dm, m.a_m, m.c_m, dn);
  last_unit(dn, m.b_n, m.c_n, dm);
  return m;
}

std::map<std::pair<int, int>, TuneShape> tune_shapes(const Dag& d) {
  std::map<std::pair<int, int>, TuneShape> out;
  for (int64_t u = d.n_leaves; u < d.n_nodes(); ++u) {
    if (d.kind[u] == HCA || is_spec(d.kind[u])) continue;   // specs always run the general kernel
    Gemm g;
    d.gemm_shape(u, &g.M, &g.N, &g.K);
    auto it = out.find({d.kind[u], d.nvec[u]});
    if (it == out.end()) {
      out[{d.kind[u], d.nvec[u]}] = {d.nt[u], g};
      continue;
    }
    TuneShape& t = it->second;
    t.nt = std::max(t.nt, (int)d.nt[u]);
    if ((double)g.M * g.N * g.K > (double)t.gemm.M * t.gemm.N * t.gemm.K) t.gemm = g;
  }
  return out;
}

void decompose(const Gemm& g, int nt, int choice, int prec, HecDesc* h, int nt_run) {
  if (choice < 0 || choice >= kNumChoices) throw std::invalid_argument("kernel choice out of range");
  if (g.M > INT32_MAX || g.N > INT32_MAX || g.K > INT32_MAX)
    throw Error(CDAG_E_INVALID, "contraction dimensions exceed 2^31");
  const int variant = choice_variant(choice);
  const int ks = k_step(prec);
  h->map_off = -1;                           // set by the caller for a contraction over index pairs
  h->M = (int32_t)g.M;
  h->N = (int32_t)g.N;
  h->K = (int32_t)g.K;
  const TileShape& ts = kTileShapes[variant_tile(variant)];
  h->nt = nt_run > 0 ? nt_run : nt;
  h->tiles_m = (h->M + ts.bm - 1) / ts.bm;
  h->tiles_n = (h->N + ts.bn - 1) / ts.bn;
  const int64_t base = (int64_t)nt * h->tiles_m * h->tiles_n;
  int64_t splits = std::min<int64_t>((kSplitTarget + base - 1) / base, h->K / kMinKSplit);
  splits = choice_split_k(choice) ? std::max<int64_t>(splits, 1) : 1;
  int64_t kspl = (h->K + splits - 1) / splits;
  kspl = (kspl + ks - 1) / ks * ks;
  splits = (h->K + kspl - 1) / kspl;
  h->splits = (int32_t)splits;
  h->k_split = (int32_t)kspl;
  h->tile_count = (int32_t)((int64_t)h->nt * h->tiles_m * h->tiles_n * splits);
}

// Cut h into the output tiles of variant v (its K splits stay).
static void retile(int v, HecDesc* h) {
  const TileShape& ts = kTileShapes[variant_tile(v)];
  h->tiles_m = (h->M + ts.bm - 1) / ts.bm;
  h->tiles_n = (h->N + ts.bn - 1) / ts.bn;
  h->tile_count = (int32_t)((int64_t)h->nt * h->tiles_m * h->tiles_n * h->splits);
}

// Every tile of one product form gives the same bits (each output adds its
// products in the same order), so without an explicit choice the tile follows
// the GEMM.  All with one LDS stage: it leaves room for more workgroups per
// compute unit, and no size measured was faster with two (FP64 K22 at N = 64
// 685 -> 623 us, FP32 K33 572 -> 502, split BF16 K22 at N = 48 337 -> 172).
// Measured (us, waves of one kind, Nt 8 to 32; N and M: the GEMM's):
//   three products (N <= 32): 32 x 32, but 64 x 32 from M = 64 on (K32 at N =
//     32: FP64 119 -> 102, FP32 68 -> 59; K22, M = 32: 130 against 184);
//   four products: from N = 65 to 80, for short K, 64 x 80 with no padded
//     column of blocks (K32 at N = 72 FP64 2148 -> 1487, FP32 1144 -> 803, at 66
//     1740 -> 1224 and 952 -> 685; K22 at 72 1991 -> 1714 and 1086 -> 929; but
//     K33, whose M = N = 72 are two of its tiles, 2400 against 2972);
//     otherwise 64 x 64, or 48 x 48 where N fills its tiles better (FP64 K33
//     at N = 72 2860 -> 2338, 96 7533 -> 5134, FP32 K22 at 96 1563 -> 1180; at
//     64 964 against 1389), to N = 64 only for long K (FP64 K33 at N = 48
//     450 -> 368; K22, K = N: FP32 at 48 240 against 279, FP64 at 45 540
//     against 620);
//   split BF16 (one form on every tile): to N = 32 as three products; to 64 the
//     64 x 64 tile (K22 at N = 48, two pieces: 172 against 207 and more); above,
//     128 x 64 with two pieces (K33 at N = 96 1467 -> 1393, 128 912 -> 774) and
//     128 x 128 with three (1443 -> 1138 at 128), which split each operand
//     value fewer times.
int default_variant(int prec, int variant, const Gemm& g) {
  const bool bf16 = prec >= 2, gauss = !bf16 && variant_tile(variant) == 1;
  if (gauss || (bf16 && g.N <= 32)) return variant_of(g.M >= 64 ? 4 : 1, 1, 1);
  if (bf16) {
    if (g.N <= 64) return variant_of(0, 1, 1);
    return prec == 2 ? variant_of(3, 1, 1) : kExtraVariantId;
  }
  if (g.N > 64 && g.N <= 80 && g.K < 512) return kExtraVariantId + kNumTiles;
  const bool fits48 = (g.N + 47) / 48 * 48 < (g.N + 63) / 64 * 64;
  return variant_of(fits48 && (g.N > 64 || g.K >= 512) ? 2 : 0, 1, 1);
}

int default_tile(int prec, int kind, int n) {
  (void)prec;
  (void)kind;
  int tile = 0;                              // 64 x 64
  if (n % 64 == 0) tile = 0;
  else if (n % 48 == 0) tile = 2;            // 48 x 48
  else if (n % 32 == 0 || n < 32) tile = 1;  // 32 x 32
  return choice_of(variant_of(tile, 1), true);
}

// decompose() for a contraction of (kind, N) without a choice: the K splits of
// default_tile(), in the tiles of default_variant().
static int decompose_default(const Gemm& g, int nt, int prec, int kind, int n, HecDesc* h, int nt_run = 0) {
  const int choice = default_tile(prec, kind, n);
  decompose(g, nt, choice, prec, h, nt_run);
  const int v = default_variant(prec, choice_variant(choice), g);
  retile(v, h);
  return v;
}

int decompose_candidate(const Gemm& g, int nt, int choice, int prec, int kind, int n, HecDesc* h) {
  if (choice == kNoChoice) return decompose_default(g, nt, prec, kind, n, h);
  decompose(g, nt, choice, prec, h);
  return choice_variant(choice);
}

int64_t store_choices(const std::map<std::pair<int, int>, TuneRow>& rows, int prec, bool uniform, TileTable* tiles) {
  // fastest choice by t(choice), or kNoChoice; -1 where nothing was timed
  auto pick = [](auto&& t, bool may_have_none) {
    int best = -1;
    for (int ch = 0; ch < kNumChoices; ++ch)
      if (t(ch) < kNotTimed && (best < 0 || t(ch) < t(best))) best = ch;
    const bool none = may_have_none && t(kNoChoice) < kNotTimed;
    return none && (best < 0 || t(kNoChoice) <= t(best)) ? (int)kNoChoice : best;
  };
  auto store = [&](const std::pair<int, int>& shape, int ch) {
    const auto key = std::make_tuple(prec, shape.first, shape.second);
    if (ch == kNoChoice) tiles->erase(key);
    else (*tiles)[key] = ch;
  };
  int64_t n = 0;
  if (!uniform) {
    for (const auto& kv : rows) {
      const int ch = pick([&](int c) { return kv.second.t[c]; }, true);
      if (ch < 0) continue;
      store(kv.first, ch);
      ++n;
    }
    return n;
  }
  if (rows.empty()) return 0;
  bool one_variant = true;
  for (const auto& kv : rows) one_variant &= kv.second.default_variant == rows.begin()->second.default_variant;
  const int ch = pick(
      [&](int c) {
        double t = 0;
        for (const auto& kv : rows) {
          if (kv.second.t[c] >= kNotTimed) return kNotTimed;
          t += kv.second.weight * kv.second.t[c];
        }
        return t;
      },
      one_variant);
  if (ch < 0) return 0;
  for (const auto& kv : rows) store(kv.first, ch);
  return (int64_t)rows.size();
}

// Descriptor (without offsets) of exterior contraction u over nt_run of its time
// slices; returns the kernel variant that runs it.  The split-K decision is the
// contraction's own (independent of batching), so results do not depend on how
// contractions are grouped into launches.
static int contraction_of(const Dag& d, int64_t u, int prec, const TileTable& tiles, int nt_run, HecDesc* h) {
  Gemm g;
  d.gemm_shape(u, &g.M, &g.N, &g.K);
  *h = HecDesc{};
  if (is_spec(d.kind[u])) {
    decompose(g, d.nt[u], choice_of(variant_of(kGenTile, 1, 2), false), prec, h, nt_run);
    return kGenVariant;
  }
  const auto it = tiles.find(std::make_tuple(prec, (int)d.kind[u], (int)d.nvec[u]));
  if (it == tiles.end()) return decompose_default(g, d.nt[u], prec, d.kind[u], d.nvec[u], h, nt_run);
  decompose(g, d.nt[u], it->second, prec, h, nt_run);
  return choice_variant(it->second);
}

std::vector<double> item_flops(const Dag& d, int prec, const TileTable& tiles) {
  std::vector<double> out(d.n_nodes(), 0.0);
  for (int64_t u = d.n_leaves; u < d.n_nodes(); ++u) {
    if (d.kind[u] == HCA) continue;
    HecDesc h;
    const int v = contraction_of(d, u, prec, tiles, d.nt[u], &h);
    const TileShape& ts = kTileShapes[v == kGenVariant ? kGenTile : variant_tile(v)];
    out[u] = 8.0 * std::min(ts.bm, h.M) * std::min(ts.bn, h.N) * h.k_split;
  }
  return out;
}

KernelPlan make_kernel_plan(const Dag& d, const Plan& p, int prec, const TileTable& tiles, bool fuse_traces) {
  KernelPlan kp;
  kp.prec = prec;
  const int64_t acc_bytes = prec == CDAG_FP64 ? 8 : 4;   // one real accumulator

  // tree index of each root, correlator buffers
  std::vector<int64_t> tree_of(d.n_nodes(), -1);
  for (int64_t t = 0; t < (int64_t)d.tree_root.size(); ++t) tree_of[d.tree_root[t]] = t;
  kp.tree_corr_off.resize(d.tree_root.size());
  int64_t co = 0;
  for (size_t t = 0; t < d.tree_root.size(); ++t) {
    kp.tree_corr_off[t] = co;
    co += 16LL * d.nt[d.tree_root[t]];
  }
  kp.corr_bytes = align256(std::max<int64_t>(co, 16));
  int32_t n_corr = 0;
  for (int32_t c : d.corr) n_corr = std::max(n_corr, c + 1);
  kp.sum_nt.assign(n_corr, 0);
  for (size_t g = 0; g < d.corr.size(); ++g) kp.sum_nt[d.corr[g]] = d.nt[d.root_of_graph[g]];
  kp.sum_corr_off.resize(n_corr);
  int64_t so = 0;
  for (int32_t c = 0; c < n_corr; ++c) {
    kp.sum_corr_off[c] = so;
    so += 16LL * kp.sum_nt[c];
  }
  kp.sums_bytes = align256(std::max<int64_t>(so, 16));

  for (int64_t u = d.n_leaves; u < d.n_nodes(); ++u)
    if (is_spec(d.kind[u]) && prec >= 2)
      throw Error(CDAG_E_INVALID, "contractions over any index pairs run in FP64 and FP32 only");
  // one index map per (spec, N), laid out after the descriptor tables
  std::map<std::pair<int32_t, int32_t>, int64_t> map_index;
  std::vector<IndexMap> maps;
  // Each contraction's descriptor (without offsets) and kernel variant, the same
  // in every pass.  A pass covers nt / t_chunks slices; the split count follows
  // the whole contraction (all nt slices), so it does not change with t_chunks
  // and the results stay bit-identical.
  std::vector<HecDesc> proto(d.n_nodes());
  std::vector<int> variant(d.n_nodes(), -1);
  for (int64_t u = d.n_leaves; u < d.n_nodes(); ++u) {
    if (d.kind[u] == HCA) continue;
    variant[u] = contraction_of(d, u, prec, tiles, (int)(d.nt[u] / p.chunks()), &proto[u]);
  }
  auto ws_of = [&](const HecDesc& h) {
    return h.splits > 1 ? align256((int64_t)h.splits * h.nt * 2 * h.M * h.N * acc_bytes) : 0;
  };

  // pass 1: workspace size (max over plan steps; an execution step with more
  // runs its split contractions in several rounds of it)
  for (const auto& step : p.steps) {
    int64_t ws = 0;
    for (int64_t u : step)
      if (d.kind[u] != HCA) ws += ws_of(proto[u]);
    kp.ws_bytes = std::max(kp.ws_bytes, ws);
  }
  // [leaf region][half 0: tensor pool, workspace][half 1 (t_chunks > 1)]...
  const int64_t C = p.chunks();
  kp.chunks = C;
  kp.half_bytes = align256(p.pool_bytes) + kp.ws_bytes;
  kp.ws_off = align256(p.leaf_region_bytes + p.pool_bytes);
  kp.tensors_end = p.leaf_region_bytes + p.halves() * kp.half_bytes;

  // pass 2: descriptors (host blob; arena offset = blob_off + host offset),
  // one set per pass over the time slices: pass k runs in half k % 2 on
  // slices [k nt / C, (k + 1) nt / C) of every tensor.
  kp.launch_off.reserve(p.n_xsteps() + 1);
  // last round (step, for traces) that an operand was counted in, per variant
  std::vector<int64_t> hec_mark[kAllVariants], hca_mark;
  int64_t round = 0, step_id = 0;
  for (int64_t k = 0; k < C; ++k) {
    const int64_t shift = (k % 2) * kp.half_bytes;
    // arena offset of operand x of a contraction in pass k: a resident leaf's
    // slices of this pass, else the planned offset in the pass's half
    auto operand_off = [&](int64_t x, int64_t planned) {
      if (p.opts.leaves_resident && d.is_leaf(x)) return p.leaf_off[x] + k * p.tsize(d, x);
      return planned + shift;
    };
    const Plan::Program& prog = p.program(k);
    for (int64_t s = 0; s < prog.n(); ++s) {
      const size_t step_first = kp.launches.size();
      kp.launch_off.push_back((int64_t)kp.launches.size());
      constexpr int kGroups = kAllVariants;
      // Launches are collected per kernel variant in rounds: a round ends where
      // its split contractions have filled the workspace, which the next one
      // then uses again.
      struct Round {
        std::vector<HecDesc> hec[kGroups];
        int64_t tiles[kGroups] = {0};
        double flops[kGroups] = {0}, bytes[kGroups] = {0};
        int32_t kinds[kGroups] = {0};
        bool ragged[kGroups] = {false};
        std::vector<RedDesc> red;
        double red_bytes = 0;
        int32_t red_kinds = 0;
        int64_t ws_used = 0, red_items = 0;
      } rd;
      auto flush_round = [&] {
        for (int tl = 0; tl < kGroups; ++tl) {
          if (rd.hec[tl].empty()) continue;
          Launch L{L_HEC, tl, (int32_t)rd.hec[tl].size(), 0, rd.tiles[tl], 0};
          L.flops = rd.flops[tl];
          L.bytes = rd.bytes[tl];
          L.kinds = rd.kinds[tl];
          L.interior = rd.ragged[tl] ? 0 : 1;
          L.host_desc = (int64_t)kp.blob.size();
          for (auto& h : rd.hec[tl]) put(kp.blob, h);
          kp.launches.push_back(L);
        }
        if (!rd.red.empty()) {
          Launch L{L_RED, 0, (int32_t)rd.red.size(), 0, rd.red_items, 0};
          L.bytes = rd.red_bytes;
          L.kinds = rd.red_kinds;
          L.host_desc = (int64_t)kp.blob.size();
          for (auto& x : rd.red) put(kp.blob, x);
          kp.launches.push_back(L);
        }
        rd = Round();
        ++round;
      };
      double hca_flops = 0, hca_bytes = 0;
      std::vector<HcaDesc> hca;
      // algorithmic bytes of a launch: each distinct operand read once, each
      // output written once (operands shared by contractions of one launch,
      // e.g. a closing meson traced against many roots, count once)
      auto operand_bytes = [&](std::vector<int64_t>& mark, int64_t id, int64_t x) {
        if (mark.empty()) mark.assign(d.n_nodes(), -1);
        if (mark[x] == id) return 0.0;
        mark[x] = id;
        return (double)p.tsize(d, x);
      };
      const int64_t hca_id = step_id++;
      for (int64_t ri = prog.off[s]; ri < prog.off[s + 1]; ++ri) {
        const PlanRec& r = prog.recs[ri];
        if (r.op != OP_EXEC) continue;
        const int64_t u = r.node;
        const double fl = d.flops(u) / (double)C;
        kp.flops += fl;
        const int64_t a_off = operand_off(d.left[u], r.a_off), b_off = operand_off(d.right[u], r.b_off);
        if (d.kind[u] == HCA) {
          HcaDesc h{};
          h.p_off = a_off;
          h.q_off = b_off;
          h.nt = (int32_t)(d.nt[u] / C);
          // relative to the correlator buffer; fixed up below (needs corr_off)
          h.out_off = -1 - (kp.tree_corr_off[tree_of[u]] + 16LL * k * h.nt);
          h.n = d.nvec[u];
          hca.push_back(h);
          hca_flops += fl;
          hca_bytes += operand_bytes(hca_mark, hca_id, d.left[u]) + operand_bytes(hca_mark, hca_id, d.right[u]);
          continue;
        }
        HecDesc h = proto[u];
        const int tl = variant[u];
        const bool gen = tl == kGenVariant;
        h.map_off = -1;
        if (gen) {
          const auto key = std::make_pair(d.kind[u], d.nvec[u]);
          auto it = map_index.find(key);
          if (it == map_index.end()) {
            it = map_index.emplace(key, (int64_t)maps.size()).first;
            maps.push_back(index_map(d.specs[d.kind[u] - kSpecBase], d.nvec[u]));
          }
          h.map_off = -2 - it->second;                   // fixed up below (needs the layout)
        }
        const int64_t ws_bytes = ws_of(h);
        if (rd.ws_used + ws_bytes > kp.ws_bytes || rd.tiles[tl] + h.tile_count > INT32_MAX) flush_round();
        const double ab = operand_bytes(hec_mark[tl], round, d.left[u]) +
                          operand_bytes(hec_mark[tl], round, d.right[u]) + (double)p.tsize(d, u);
        kp.hec_flops += fl;
        kp.hec_bytes += ab;
        rd.flops[tl] += fl;
        rd.bytes[tl] += ab;
        rd.kinds[tl] |= 1 << std::min<int32_t>(d.kind[u], 7);
        h.a_off = a_off;
        h.b_off = b_off;
        h.c_off = r.dev_off + shift;
        h.ws_off = -1;
        h.tile_begin = (int32_t)rd.tiles[tl];
        rd.tiles[tl] += h.tile_count;
        if (gen || !hec_interior(h, kTileShapes[variant_tile(tl)].bm, kTileShapes[variant_tile(tl)].bn, k_step(prec)))
          rd.ragged[tl] = true;
        kp.hec_items += h.tile_count;
        if (h.splits > 1) {
          h.ws_off = kp.ws_off + shift + rd.ws_used;
          RedDesc e{};
          e.ws_off = h.ws_off;
          e.c_off = h.c_off;
          e.mn = h.M * h.N;
          e.nt = h.nt;
          e.splits = h.splits;
          e.item_begin = (int32_t)rd.red_items;
          rd.red_items += red_items(e.nt, e.mn);
          rd.red.push_back(e);
          rd.red_bytes += 2.0 * e.nt * (double)e.mn * ((double)e.splits * acc_bytes + elem_bytes_of(prec));
          rd.red_kinds |= 1 << d.kind[u];
          rd.ws_used += ws_bytes;
        }
        rd.hec[tl].push_back(h);
      }
      flush_round();
      if (!hca.empty()) {
        int64_t n_titems = 0;
        for (auto& h : hca) { h.item_begin = (int32_t)n_titems; n_titems += h.nt; }
        // the exterior-contraction launch of this step that carries the
        // traces, if fused: the last one of one workgroup per item whose grid
        // stays within kMaxGrid with the trace workgroups added
        Launch* carrier = nullptr;
        for (size_t li = kp.launches.size(); fuse_traces && li-- > step_first;) {
          Launch& L = kp.launches[li];
          if (L.type != L_HEC || L.tile == kGenVariant || variant_grid(L.tile) != 1) continue;
          if (L.n_items + trace_blocks(kTileShapes[variant_tile(L.tile)].nth, n_titems) > kMaxGrid) continue;
          carrier = &L;
          break;
        }
        if (carrier) {
          carrier->tr_n_desc = (int32_t)hca.size();
          carrier->tr_n_items = n_titems;
          carrier->tr_flops = hca_flops;
          carrier->tr_bytes = hca_bytes;
          carrier->kinds |= 1 << HCA;
          carrier->tr_host_desc = (int64_t)kp.blob.size();
          for (auto& h : hca) put(kp.blob, h);
        } else {
          Launch L{L_HCA, 0, (int32_t)hca.size(), 0, n_titems, 0};
          L.flops = hca_flops;
          L.bytes = hca_bytes;
          L.kinds = 1 << HCA;
          L.host_desc = (int64_t)kp.blob.size();
          for (auto& h : hca) put(kp.blob, h);
          kp.launches.push_back(L);
        }
      }
    }
  }
  kp.launch_off.push_back((int64_t)kp.launches.size());

  // cross-diagram sums: per correlator, entries in ascending graph order
  std::vector<std::vector<int64_t>> by_corr(n_corr);
  for (size_t g = 0; g < d.corr.size(); ++g) by_corr[d.corr[g]].push_back((int64_t)g);
  std::vector<XsumDesc> xd;
  std::vector<XsumEntry> xe;
  int64_t xitems = 0;
  for (int32_t c = 0; c < n_corr; ++c) {
    XsumDesc x{};
    x.out_off = kp.sum_corr_off[c];   // relative; fixed up below
    x.e_begin = (int32_t)xe.size();
    for (int64_t g : by_corr[c])
      xe.push_back({kp.tree_corr_off[tree_of[d.root_of_graph[g]]], d.w_re[g], d.w_im[g]});
    x.e_end = (int32_t)xe.size();
    x.nt = kp.sum_nt[c];
    x.item_begin = (int32_t)xitems;   // a correlator without graphs (nt 0) has no items
    xitems += x.nt;
    xd.push_back(x);
  }
  while (kp.blob.size() % 16) kp.blob.push_back(0);
  kp.xsum = {L_XSUM, 0, (int32_t)xd.size(), 0, xitems, (int64_t)kp.blob.size()};
  for (auto& x : xd) put(kp.blob, x);
  const int64_t entries_host = (int64_t)kp.blob.size();
  for (auto& e : xe) put(kp.blob, e);
  while (kp.blob.size() % 16) kp.blob.push_back(0);
  const int64_t maps_host = (int64_t)kp.blob.size();
  for (auto& m : maps) put(kp.blob, m);

  // final layout and fix-ups of buffer-relative offsets
  kp.blob_off = align256(kp.tensors_end);
  kp.corr_off = align256(kp.blob_off + (int64_t)kp.blob.size());
  kp.sums_off = kp.corr_off + kp.corr_bytes;
  kp.total_bytes = align256(kp.sums_off + kp.sums_bytes);
  for (Launch& L : kp.launches) {
    L.desc_off = kp.blob_off + L.host_desc;
    if (L.type == L_HEC && L.tile == kGenVariant) {
      auto* h = reinterpret_cast<HecDesc*>(kp.blob.data() + L.host_desc);
      for (int32_t i = 0; i < L.n_desc; ++i)
        h[i].map_off = kp.blob_off + maps_host + (-2 - h[i].map_off) * (int64_t)sizeof(IndexMap);
    }
    if (L.type == L_HCA) {
      auto* h = reinterpret_cast<HcaDesc*>(kp.blob.data() + L.host_desc);
      for (int32_t i = 0; i < L.n_desc; ++i) h[i].out_off = kp.corr_off + (-1 - h[i].out_off);
    }
    if (L.tr_n_desc > 0) {
      L.tr_desc_off = kp.blob_off + L.tr_host_desc;
      auto* h = reinterpret_cast<HcaDesc*>(kp.blob.data() + L.tr_host_desc);
      for (int32_t i = 0; i < L.tr_n_desc; ++i) h[i].out_off = kp.corr_off + (-1 - h[i].out_off);
    }
  }
  kp.xsum.desc_off = kp.blob_off + kp.xsum.host_desc;
  kp.xsum_entries_off = kp.blob_off + entries_host;
  auto* x = reinterpret_cast<XsumDesc*>(kp.blob.data() + kp.xsum.host_desc);
  for (int32_t i = 0; i < kp.xsum.n_desc; ++i) x[i].out_off += kp.sums_off;
  auto* e = reinterpret_cast<XsumEntry*>(kp.blob.data() + entries_host);
  for (size_t i = 0; i < xe.size(); ++i) e[i].root_off += kp.corr_off;
  return kp;
}

}  // namespace cdag
