"""Performance cases of the contraction-DAG engine: whole executes through the
public entry points (build_cdag, schedule, set_mem_budget, execute,
fetch_correlators, cdag_fetch_sums), from the smallest DAG, where latency and
launches count, to the baryon DAG with its leaves uploaded inside the step.

One pass is what a program does per configuration: execute the planned DAG and
fetch every correlator and the cross-diagram sums.  FP64 passes return them in
complex128, the other precisions (complex64 storage) in complex64.

A case holds plain values:
  shape       ring (meson traces), perm (four-meson permutation traces), chain
              (baryon chains), mix (rings and chains over families of N),
              rank4 (rank-4 intermediates), pairs (contractions over any index
              pairs with permuted outputs)
  n, nt       distillation vectors N (mix: unused), time slices
  mesons, baryons, graphs, graph_seed   leaves, graphs and the seed of the
              graphs' structure (the tensors' values come from prepare's seed)
  prec        fp64, fp32, bf16x3, bf16x6;  c64: leaves given in complex64
  batched     waves of ready contractions, or one contraction per step
  resident    leaves kept on the device, or uploaded in every pass
  lookahead   of the wave cut (-1: every ready contraction);  chunks: passes
              over the time slices;  issue: 0 eager, 1 and 2 replayed graphs
  budget      bytes of device memory, 0 for unlimited, -1 for a quarter of the
              input order's live peak
  choice      kernel choice "tile.grid.stages.split" kept from an earlier
              tuning, or "" for the library's defaults
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

K22, K32, K33, HCA, C1, C2, C3 = 0, 1, 2, 3, 4, 5, 6
SPEC_BASE = 16
SUMMED = {K22: 1, K32: 1, K33: 2, C1: 1, C2: 2, C3: 3}
FAMILIES = (32, 48, 64, 96, 128)      # the N of a mixed batch
ALL_READY = (1 << 63) - 1

# (rank_l, rank_r, pairs, perm): contractions over other index pairs, with
# permuted outputs
SPECS = (
    (3, 2, ((0, 1),), (2, 0, 1)),
    (3, 3, ((2, 0), (0, 2)), (1, 0)),
    (2, 2, ((0, 0),), (1, 0)),
    (4, 3, ((1, 0), (3, 2)), (0, 2, 1)),
    (3, 3, ((1, 1),), (3, 1, 0, 2)),
)

_BASE = dict(shape="ring", n=64, nt=32, mesons=16, baryons=0, graphs=100, graph_seed=1, prec="fp64", c64=False,
             batched=True, resident=False, lookahead=-1, chunks=1, issue=1, budget=0, choice="")


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # the smallest call: four small mesons, six permutation traces, every option at its default
        _case(name="perm_n16", shape="perm", n=16, nt=8, mesons=4, graphs=6, lookahead=0),
        # a short queue run one contraction per step, as the paper's runtime does
        _case(name="ring_n32_queue", n=32, nt=8, mesons=8, graphs=40, graph_seed=2, batched=False, lookahead=0,
              resident=True),
        # the meson configuration with its leaves on the device, kernel choices kept from a tuning
        _case(name="ring_n64_fp64", graphs=2000, graph_seed=3, resident=True, choice="5.1.1.0"),
        # one small-N family of the batched configuration
        _case(name="ring_n48_fp32", n=48, nt=64, mesons=8, graphs=600, graph_seed=4, prec="fp32", c64=True,
              resident=True),
        # a basis size that no tile divides, odd time extent
        _case(name="ring_n45_fp64", n=45, nt=21, mesons=12, graphs=400, graph_seed=5, resident=True),
        # the meson configuration in memory a quarter of its live peak, passes over the time slices
        _case(name="ring_n64_budget", graphs=2000, graph_seed=3, lookahead=384, chunks=16, budget=-1,
              choice="5.1.1.0"),
        # the baryon configuration: 32e9 bytes, leaves from the host in every step, kernel choices kept from a tuning
        _case(name="chain_n64_headline", shape="chain", mesons=12, baryons=12, graphs=500, graph_seed=6, chunks=8,
              issue=0, budget=32 * 10**9, choice="5.1.1.0"),
        # baryon chains with the leaves on the device, in single precision and in split BF16
        _case(name="chain_n64_fp32", shape="chain", nt=16, mesons=6, baryons=6, graphs=200, graph_seed=7, prec="fp32",
              c64=True, resident=True),
        _case(name="chain_n72_bf16x3", shape="chain", n=72, nt=12, mesons=6, baryons=6, graphs=150, graph_seed=8,
              prec="bf16x3", c64=True, resident=True),
        # mixed rank and N in one batch, under a budget
        _case(name="mix_fp32", shape="mix", n=0, nt=8, mesons=6, baryons=4, graphs=600, graph_seed=9, prec="fp32",
              c64=True, issue=0, chunks=2, budget=8 * 10**9),
        # three-baryon systems: rank-4 intermediates
        _case(name="rank4_n24_fp64", shape="rank4", n=24, nt=4, mesons=4, baryons=6, graphs=60, graph_seed=10,
              resident=True),
        # contractions over any index pairs
        _case(name="pairs_n20_fp64", shape="pairs", n=20, nt=4, mesons=5, baryons=5, graphs=60, graph_seed=11,
              resident=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case over the same ranges: every shape, N from the smallest to
    the largest of its kind (multiples of 8 and not), odd time extents, every
    precision and issue mode, leaves resident or not, tuned or default
    kernels."""
    while True:
        shape = rng.choice(("ring", "ring", "perm", "chain", "chain", "mix", "rank4", "pairs"))
        top = {"ring": 128, "perm": 64, "chain": 96, "rank4": 32, "pairs": 28, "mix": 0}[shape]
        n = _log_int(rng, 8, top) if top else 0
        if top and rng.random() < 0.5:
            n = min(top, max(8, (n + 4) // 8 * 8))
        nt = rng.choice((8, 12, 16)) if shape == "mix" else _log_int(rng, 1, 32)
        # split BF16 takes the named and general kinds, not other index pairs
        prec = rng.choice(("fp64", "fp64", "fp32") if shape == "pairs" else
                          ("fp64", "fp64", "fp64", "fp32", "fp32", "bf16x3", "bf16x6"))
        batched = rng.random() < 0.9
        chunks = rng.choice([c for c in (1, 1, 1, 2, 4, 8) if nt % c == 0])
        tile = rng.choice(("", "", "", "0.1.1.0", "1.1.2.1", "3.1.1.0", "4.1.1.0", "5.1.1.0", "5.1.2.1"))
        c = _case(shape=shape, n=n, nt=nt,
                  mesons=4 if shape == "perm" else rng.randrange(6, 17),
                  baryons=rng.randrange(4, 7) if shape in ("chain", "mix", "rank4", "pairs") else 0,
                  graphs=rng.randrange(4, 20) if shape == "perm" else _log_int(rng, 20, 80 if not batched else 800),
                  graph_seed=rng.randrange(1 << 20), prec=prec, c64=prec != "fp64" or rng.random() < 0.2,
                  batched=batched, resident=rng.random() < 0.6, lookahead=rng.choice((0, 16, -1)) if batched else 0,
                  chunks=chunks, issue=rng.choice((0, 1, 1, 2)),
                  budget=-1 if shape == "ring" and rng.random() < 0.2 else 0, choice=tile)
        w = work(c)
        # within the listed cases: time of a pass and bytes of the leaves
        if w["flops"] <= (2e12 if shape in ("ring", "chain", "mix") else 4e10) and w["bytes"] <= 1.2e9:
            return c


# ---------------------------------------------------------------- graphs
def _shapes(case):
    """[(rank, N)] of the leaves."""
    if case["shape"] == "mix":
        return [(r, n) for n in FAMILIES for r, k in ((2, case["mesons"]), (3, case["baryons"])) for _ in range(k)]
    n = case["n"]
    r4 = 2 if case["shape"] in ("rank4", "pairs") else 0
    return [(2, n)] * case["mesons"] + [(3, n)] * case["baryons"] + [(4, n)] * r4


def _ring(r, mes, lmin, lmax):
    """tr(A_1 .. A_L) over distinct leaves as a random binary tree."""
    seq = r.sample(mes, r.randint(lmin, min(lmax, len(mes))))
    ops = []

    def product(s):
        if len(s) == 1:
            return s[0]
        k = r.randrange(1, len(s))
        left, right = product(s[:k]), product(s[k:])
        ops.append((K22, left, right))
        return -len(ops)

    cut = r.randrange(1, len(seq))
    p, q = product(seq[:cut]), product(seq[cut:])
    ops.append((HCA, p, q))
    return ops


def _chain(r, bar, mes):
    a, c = r.sample(bar, 2)
    b, d = r.sample(mes, 2)
    return [(K32, a, b), (K33, -1, c), (HCA, -2, d)]


def _rank4(r, bar, mes, r4):
    b, m, x = r.sample(bar, 4), r.sample(mes, 2), r.choice(r4)
    return r.choice((
        [(C1, b[0], b[1]), (C2, -1, b[2]), (K33, -2, b[3]), (HCA, -3, m[0])],
        [(C1, b[0], b[1]), (C3, -1, x), (HCA, -2, m[0])],
        [(C1, m[0], b[0]), (K33, -1, b[1]), (HCA, -2, m[1])],
        [(C2, x, m[0]), (HCA, -1, m[1])],
    ))


def _pairs(r, bar, mes, r4):
    b, m, x = r.sample(bar, 4), r.sample(mes, 3), r.choice(r4)
    S = [SPEC_BASE + i for i in range(len(SPECS))]
    return r.choice((
        [(S[0], b[0], m[0]), (S[1], -1, b[1]), (HCA, -2, m[1])],
        [(S[2], m[0], m[1]), (HCA, -1, m[2])],
        [(S[1], b[0], b[1]), (S[2], m[0], m[1]), (HCA, -1, -2)],
        [(S[3], x, b[0]), (S[1], -1, b[1]), (HCA, -2, m[0])],
        [(C1, b[0], b[1]), (C2, -1, b[2]), (K33, -2, b[3]), (HCA, -3, m[0])],
        [(S[4], b[0], b[1]), (C2, -1, m[0]), (HCA, -2, m[1])],
    ))


def _graphs(case):
    """[(ops, correlator, weight)]."""
    r = random.Random(case["graph_seed"])
    shapes = _shapes(case)

    def ids(rank, n):
        return [i for i, s in enumerate(shapes) if s == (rank, n)]

    out, shape = [], case["shape"]
    for g in range(case["graphs"]):
        n = FAMILIES[g % len(FAMILIES)] if shape == "mix" else case["n"]
        mes, bar, r4 = ids(2, n), ids(3, n), ids(4, n)
        corr = r.randrange(4)
        if shape == "mix":
            ops = _ring(r, mes, 4, 6) if g // len(FAMILIES) % 2 == 0 else _chain(r, bar, mes)
            corr += 4 * (g % len(FAMILIES))
        elif shape == "ring":
            ops = _ring(r, mes, 4, 8)
        elif shape == "perm":
            p = r.sample(mes, 4)
            ops = [(K22, p[0], p[1]), (K22, p[2], p[3]), (HCA, -1, -2)]
        elif shape == "chain":
            ops = _chain(r, bar, mes)
        elif shape == "rank4":
            ops = _rank4(r, bar, mes, r4)
        else:
            ops = _pairs(r, bar, mes, r4)
        out.append((ops, corr, r.choice((-1.0, 1.0))))
    return out


def _merged(case):
    """The DAG with equal sub-trees merged: ([(kind, left, right)] by node id
    after the leaves, root of each graph, {leaf or node: (rank, N)})."""
    dims = dict(enumerate(_shapes(case)))
    nodes, seen, roots = [], {}, []
    for ops, _, _ in _graphs(case):
        at = []
        for kind, a, b in ops:
            key = (kind, a if a >= 0 else at[-a - 1], b if b >= 0 else at[-b - 1])
            if key not in seen:
                u = seen[key] = len(dims)
                nodes.append(key)
                (rl, n), (rr, _) = dims[key[1]], dims[key[2]]
                c = 2 if kind == HCA else len(SPECS[kind - SPEC_BASE][2]) if kind >= SPEC_BASE else SUMMED[kind]
                dims[u] = (rl + rr - 2 * c, n)
            at.append(seen[key])
        roots.append(at[-1])
    return nodes, roots, dims


def work(case):
    """Each leaf read once, each correlator and sum written once; 8 flops per
    complex multiply-add of the merged DAG."""
    nodes, roots, dims = _merged(case)
    nt = case["nt"]
    flops = 0.0
    for kind, a, b in nodes:
        rl, rr, ro = dims[a][0], dims[b][0], (0 if kind == HCA else dims[a][0] + dims[b][0])
        c = 2 if kind == HCA else len(SPECS[kind - SPEC_BASE][2]) if kind >= SPEC_BASE else SUMMED[kind]
        flops += 8.0 * nt * float(dims[a][1]) ** (rl + rr - c)
    used = {x for _, a, b in nodes for x in (a, b)}
    item = 16 if case["prec"] == "fp64" else 8
    bytes_ = sum(float(n) ** r * nt * item for i, (r, n) in enumerate(_shapes(case)) if i in used)
    n_corr = 1 + max(c for _, c, _ in _graphs(case))
    return {"bytes": bytes_ + 16.0 * nt * (len(set(roots)) + n_corr), "flops": flops}


# ---------------------------------------------------------------- tensors
def _tensors(case, seed):
    """The leaves on the device, complex [nt][N]..: re and im iid normal with
    deviation 1/sqrt(N) for rings and 1/N otherwise, as N-vector hadron nodes
    normalised so that products keep their scale."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float32 if case["c64"] else torch.float64
    for rank, n in _shapes(case):
        sigma = n ** -0.5 if case["shape"] in ("ring", "perm") else 1.0 / n
        x = torch.randn((case["nt"],) + (n,) * rank + (2,), dtype=real, device="cuda", generator=gen)
        yield torch.view_as_complex(x.mul_(sigma))


def prepare(case, seed):
    import paper_2511_02257_amd as X
    from paper_2511_02257_amd.device import DeviceRunner

    leaves = [SimpleNamespace(rank=r, nvec=n, nt=case["nt"], data=t.cpu().numpy())
              for (r, n), t in zip(_shapes(case), _tensors(case, seed))]
    graphs = [SimpleNamespace(ops=ops, corr=c, w=w) for ops, c, w in _graphs(case)]
    specs = [SimpleNamespace(rank_l=a, rank_r=b, pairs=p, perm=q) for a, b, p, q in SPECS]
    ctx = X.Context()
    ctx.build_cdag(leaves, graphs, specs if case["shape"] == "pairs" else ())
    budget = case["budget"] or None
    if case["budget"] == -1:
        _, _, peak = ctx.memsim(ctx.schedule("input"), 16 if case["prec"] == "fp64" else 8)
        # a step holds two operands and an output: never below four of the largest leaf
        largest = max(n ** r for r, n in _shapes(case)) * case["nt"] * (16 if case["prec"] == "fp64" else 8)
        budget = max(peak // 4, 4 * largest)
    ctx.schedule("tree")
    ctx.set_mem_budget(budget)
    ctx.set_options(leaves_resident=case["resident"], use_graphs=case["issue"],
                    wave_lookahead=ALL_READY if case["lookahead"] < 0 else case["lookahead"])
    ctx.set_time_chunks(case["chunks"])
    if case["choice"]:
        for n in {n for _, n in _shapes(case)}:
            for kind in (K22, K32, K33, C1, C2, C3):
                ctx.set_tile(case["prec"], kind, n, *map(int, case["choice"].split(".")))
    runner = DeviceRunner(ctx, 0)
    runner.ensure_arena(ctx.plan(case["prec"], case["batched"])["arena_bytes"])
    return SimpleNamespace(ctx=ctx, runner=runner, prec=case["prec"], batched=case["batched"])


def run(state):
    state.runner.run(state.prec, state.batched)
    corr = np.concatenate(state.ctx.fetch_correlators())
    sums = np.concatenate(state.ctx.fetch_sums())
    if state.prec != "fp64":
        corr, sums = corr.astype(np.complex64), sums.astype(np.complex64)
    return {"correlators": corr, "sums": sums}


def _contract(kind, x, y):
    """One contraction in complex128, batched over the time slices."""
    nt, n = x.shape[0], x.shape[1]
    if kind >= SPEC_BASE:
        rl, rr, pairs, perm = SPECS[kind - SPEC_BASE]
        fl = [i for i in range(rl) if i not in [p for p, _ in pairs]]
        fr = [i for i in range(rr) if i not in [q for _, q in pairs]]
        x = x.permute([0] + [1 + i for i in fl] + [1 + p for p, _ in pairs]).contiguous()
        y = y.permute([0] + [1 + q for _, q in pairs] + [1 + i for i in fr]).contiguous()
        c = len(pairs)
    else:
        rl, rr, c, perm = x.dim() - 1, y.dim() - 1, SUMMED[kind], None
    o = torch.matmul(x.reshape(nt, n ** (rl - c), n ** c), y.reshape(nt, n ** c, n ** (rr - c)))
    o = o.reshape((nt,) + (n,) * (rl + rr - 2 * c))
    return o if perm is None else o.permute([0] + [1 + q for q in perm]).contiguous()


def exact(case, seed):
    nodes, roots, _ = _merged(case)
    val = {i: t.to(torch.complex128) for i, t in enumerate(_tensors(case, seed))}
    n_leaves = len(val)
    last = {x: i for i, (_, a, b) in enumerate(nodes) for x in (a, b)}
    out = {}
    for i, (kind, a, b) in enumerate(nodes):
        if kind == HCA:
            out[n_leaves + i] = (val[a] * val[b].transpose(1, 2)).sum((1, 2)).cpu().numpy()
        else:
            val[n_leaves + i] = _contract(kind, val[a], val[b])
        for x in {a, b}:
            if last[x] == i:
                del val[x]
    corr = [out[u] for u in roots]
    sums = {}
    for (_, c, w), v in zip(_graphs(case), corr):
        sums[c] = sums.get(c, 0) + w * v
    return {"correlators": np.concatenate(corr), "sums": np.concatenate([sums[c] for c in sorted(sums)])}
