"""The measured cases: what a user of this solver has it do, through the
binding's public entry points (``paper_1905_11722_amd/rcdp.py``).

A case names a graph shape with its sizes, how its costs are counted, a
family, an objective, a budget and a call:

* ``plan``: everything from a host graph: hand it over, build the family,
  solve, trace the schedule (``rcdp.solve_graph``);
* ``step``: the same from a graph that is on the device already;
* ``sweep``: on a family that is kept, the smallest feasible budget, then
  ``budgets`` budgets from it to 2 M(V) in one batch, each traced;
* ``dual`` / ``dual_noalloc``: on a family that is kept, the memory-indexed
  solve with its schedule;
* ``dominance``: on a family that is kept, the solve with the dominance
  skip, traced;
* ``table``: on a family that is kept, a solve and its whole (m, optarg)
  table.

The seed draws the costs, never the structure: T_v and M_v of the synthetic
graphs from their ranges, and of the CNN shapes a few per cent around the
counted FLOPs (an operator's measured time varies) or the counted activation
sizes (an allocator rounds), so inputs of another seed are another problem of
the same size.
"""

import random

import numpy as np

from paper_1905_11722_amd import rcdp, workloads

# ------------------------------------------------------------------- graphs


def _structure(c):
    kind = c["graph"]
    if kind == "chain":
        return workloads.chain(c["nodes"], 0)
    if kind == "ladder":
        return workloads.ladder(c["length"], 0)
    if kind == "layered":
        return workloads.layered(c["layers"], c["width"], c["structure"])
    if kind == "random":
        return workloads.random_dag(c["nodes"], c["p"], c["structure"])
    if kind == "resnet50":
        return workloads.resnet50(c["batch"], c["image"])
    if kind == "densenet121":
        return workloads.densenet121(c["batch"], c["image"])
    return workloads.unet(c["batch"], c["image"], depth=c["depth"])


CNN = ("resnet50", "densenet121", "unet")


def _graph(c, seed):
    """The case's graph with costs drawn from the seed."""
    g = _structure(c)
    rng = random.Random(seed)
    if c["graph"] not in CNN:
        tmax, mmax = (10, 8) if c["graph"] in ("chain", "random") else (100, 64)
        T = [rng.randint(1, tmax) for _ in range(g.n)]
        M = [rng.randint(1, mmax) for _ in range(g.n)]
    elif c["costs"] == "t10":       # the paper's convention: T is fixed, sizes vary
        g = workloads.paper_costs(g)
        T = list(g.T)
        M = [max(1, round(m * rng.uniform(0.95, 1.05))) for m in g.M]
    else:
        T = [max(1, round(t * rng.uniform(0.95, 1.05))) for t in g.T]
        M = list(g.M)
    if c["unit"] == "KiB":          # sizes in KiB: budgets beyond 16 bits
        M = [1024 * m - rng.randrange(1024) for m in M]
    return workloads.Graph(g.n, [list(x) for x in g.succ], T, M, list(g.names), list(g.ops))


def _budget(c, g):
    """The case's budget, absolute or as a share of M(V)."""
    return c["B"] if c["B"] else int(c.get("share", 1.0) * sum(g.M))


# -------------------------------------------------------------------- cases


def _case(name, call, graph, B, mode="pruned", objective="tc", costs="flops", unit="MiB", **sizes):
    c = {"call": call, "graph": graph, "mode": mode, "objective": objective, "B": B,
         "costs": costs, "unit": unit}
    c.update(sizes)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest problem: a 16-node chain; all of it is launches and waits
        _case("chain16", "plan", "chain", 64, "exact", nodes=16),
        # a branching network of 40 operators planned exactly (241 sets)
        _case("ladder40", "step", "ladder", 1024, "exact", length=20),
        # an exact family of thousands of sets in wide levels (6199 sets)
        _case("layered36", "step", "layered", 2048, "exact", layers=6, width=6, structure=0),
        # one network planned from its host graph, FLOP costs
        _case("resnet50", "plan", "resnet50", 4096, batch=32, image=224),
        # the benchmark's step, the largest table (55 M cells, 9.3e9 relaxations)
        _case("densenet121", "step", "densenet121", 4096, batch=32, image=224),
        # the same graph with the paper's costs: many sets, rows of about 1500 cells
        _case("densenet121_t10", "step", "densenet121", 4096, costs="t10", batch=32, image=224),
        # few sets, rows of up to 2.4 M cells
        _case("unet", "step", "unet", 16384, batch=8, image=572, depth=4),
        # sizes counted in KiB: 32-bit cells
        _case("resnet50_kib", "step", "resnet50", 4096 << 10, unit="KiB", batch=32, image=224),
        # the memory-centric sweep of 32 budgets on one family
        _case("resnet50_sweep", "sweep", "resnet50", 0, objective="mc", budgets=32, batch=32,
              image=224),
        # the memory-indexed solve with its schedule
        _case("densenet121_dual", "dual", "densenet121", 4096, batch=32, image=224),
        # the dominance skip on long rows
        _case("unet_dominance", "dominance", "unet", 16384, batch=8, image=572, depth=4),
        # the whole time-memory table of a network with the paper's costs
        _case("resnet50_t10_table", "table", "resnet50", 4096, costs="t10", batch=32, image=224),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the listed ranges: exact families of small graphs and
    pruned families of CNN shapes, every call, both objectives, budgets from
    tight to loose, odd sizes."""
    shape = rng.choice(("chain", "ladder", "layered", "random", "resnet50", "densenet121", "unet"))
    objective = rng.choice(("tc", "mc"))
    if shape in CNN:
        mode, costs = "pruned", rng.choice(("flops", "flops", "t10"))
        unit = rng.choice(("MiB", "MiB", "KiB")) if shape != "densenet121" else "MiB"
        if shape == "unet":
            sizes = {"batch": rng.randint(2, 8), "image": rng.randint(400, 572),
                     "depth": rng.randint(3, 4)}
        else:
            sizes = {"batch": _log(rng, 4, 24), "image": rng.randint(160, 224)}
    else:
        mode, costs, unit = rng.choice(("exact", "exact", "pruned")), "flops", "MiB"
        sizes = {"chain": {"nodes": _log(rng, 8, 160)},
                 "ladder": {"length": _log(rng, 6, 40)},
                 "layered": {"layers": rng.randint(4, 8), "width": rng.randint(2, 5),
                             "structure": rng.randrange(1 << 20)},
                 "random": {"nodes": rng.randint(8, 22), "p": round(rng.uniform(0.2, 0.5), 3),
                            "structure": rng.randrange(1 << 20)}}[shape]
    calls = ["plan", "step", "step", "sweep", "dual", "dominance", "table"]
    if unit == "KiB":               # the skip takes 16-bit cells, the dual table rows of M(V)
        calls = ["plan", "step", "step"]
    elif shape in CNN and costs == "flops":
        calls = ["plan", "step", "step", "sweep", "dual", "dominance"]
    call = rng.choice(calls)
    if call == "dual" and shape != "densenet121" and rng.random() < 0.5:
        call = "dual_noalloc"
    c = _case(None, call, shape, 0, mode, objective, costs, unit, **sizes)
    if call == "sweep":
        c["budgets"] = _log(rng, 3, 12)
        c["objective"] = "mc"
    elif call == "dominance":
        c["objective"] = "tc"
    # budgets from a little over the smallest feasible one to the loosest
    lo, hi = ((0.55, 1.5) if shape in CNN else
              (1.0, 2.0) if shape in ("chain", "ladder") else (1.8, 2.4))
    c["share"] = round(rng.uniform(lo, hi), 3)
    return c


# ---------------------------------------------------------------- the calls


def prepare(case, seed):
    g = _graph(case, seed)
    s = {"case": case, "graph": g, "B": _budget(case, g), "handle": None, "family": None}
    if case["call"] != "plan":
        s["handle"] = rcdp.Graph.create(g)
    if case["call"] not in ("plan", "step"):
        s["family"] = s["handle"].build_family(case["mode"])
    return s


def _padded(chain, n):
    """The chain in an array of the longest a chain of n nodes can be."""
    out = np.full(n, -1, dtype=np.int32)
    out[:len(chain)] = chain
    return out


def _schedule(sched, out):
    if sched is not None:
        out["chain"], out["seg"], out["cached"] = (_padded(sched.chain, len(sched.seg)),
                                                   sched.seg, sched.cached)
        out["overhead"], out["peak"], out["cache_mem"] = (sched.overhead, sched.peak,
                                                          sched.cache_mem)
    return out


def run(state):
    c = state["case"]
    call, B, objective = c["call"], state["B"], c["objective"]
    if call == "plan":
        g, fam, sol, sched = rcdp.solve_graph(state["graph"], c["mode"], B, objective)
        out = _schedule(sched, {"t": sol.t_star, "m": sol.m_star})
        sol.free()
        fam.free()
        g.free()
        return out
    if call == "step":
        fam = state["handle"].build_family(c["mode"])
        sol = fam.solve(B, objective)
        sched = sol.reconstruct() if sol.feasible else None
        out = _schedule(sched, {"t": sol.t_star, "m": sol.m_star})
        sol.free()
        fam.free()
        return out
    fam = state["family"]
    if call == "sweep":
        b_min = fam.min_budget()
        top = 2 * sum(state["graph"].M)
        n = c["budgets"]
        budgets = [b_min + (j * (top - b_min)) // (n - 1) for j in range(n)]
        sols = [sol for _, sol in fam.sweep(budgets, objective)]
        scheds = [sol.reconstruct() for sol in sols]
        out = {"b_min": b_min, "t": np.array([sol.t_star for sol in sols]),
               "m": np.array([sol.m_star for sol in sols]),
               "chain": np.stack([_padded(x.chain, len(x.seg)) for x in scheds]),
               "seg": np.stack([x.seg for x in scheds]),
               "cached": np.stack([x.cached for x in scheds]),
               "overhead": np.array([x.overhead for x in scheds]),
               "peak": np.array([x.peak for x in scheds]),
               "cache_mem": np.array([x.cache_mem for x in scheds])}
        for sol in sols:
            sol.free()
        return out
    if call == "dual":
        t, m, _, sched = fam.solve_dual(B, objective, schedule=True)
        return _schedule(sched, {"t": t, "m": m})
    if call == "dual_noalloc":
        t, m, sched = fam.solve_dual_noalloc(B, objective)
        return _schedule(sched, {"t": t, "m": m})
    if call == "dominance":
        sol = fam.solve_dominance(B)
        sched = sol.reconstruct() if sol.feasible else None
        out = _schedule(sched, {"t": sol.t_star, "m": sol.m_star})
        sol.free()
        return out
    sol = fam.solve(B, objective)
    m, arg = sol.table()
    out = {"t": sol.t_star, "m": sol.m_star, "table": m, "optarg": arg}
    sol.free()
    return out


# ------------------------------------------- what the work is, and its result


def _family(g, mode):
    """Lower sets as Python integers, by size then value."""
    pred = [0] * g.n
    for v in range(g.n):
        for w in g.succ[v]:
            pred[w] |= 1 << v
    full = (1 << g.n) - 1
    sets = {0, full}
    if mode == "pruned":
        anc, todo = {}, list(range(g.n))
        while todo:
            v = todo[-1]
            ps = [p for p in range(g.n) if pred[v] >> p & 1]
            left = [p for p in ps if p not in anc]
            if left:
                todo += left
                continue
            todo.pop()
            x = 1 << v
            for p in ps:
                x |= anc[p]
            anc[v] = x
        sets |= set(anc.values())
    else:
        level = {0}
        while level:
            level = {S | 1 << v for S in level for v in range(g.n)
                     if not S >> v & 1 and not pred[v] & ~S}
            sets |= level
    return sorted(sets, key=lambda S: (bin(S).count("1"), S)), pred


def _nodes(S):
    out = []
    while S:
        b = S & -S
        out.append(b.bit_length() - 1)
        S ^= b
    return out


class _Model:
    """Family, boundaries and sums of one graph (Section 2 and Eq. 2)."""

    def __init__(self, g, mode):
        self.g = g
        self.sets, pred = _family(g, mode)
        succ = [sum(1 << w for w in set(g.succ[v])) for v in range(g.n)]
        self.T, self.M = g.T, g.M
        self.bd, self.A, self.w = [], [], []
        for L in self.sets:
            nodes = _nodes(L)
            b = sum(1 << v for v in nodes if succ[v] & ~L)
            out = 0
            for v in nodes:
                out |= succ[v] & ~L
            back = 0
            for v in _nodes(out):
                back |= pred[v] & ~L
            self.bd.append(b)
            self.A.append(self.sum(self.M, out) + self.sum(self.M, back))
            self.w.append(self.sum(self.T, L & ~b) + 1)

    @staticmethod
    def sum(c, S):
        return sum(c[v] for v in _nodes(S))

    def member(self):
        return np.array([[S >> v & 1 for v in range(self.g.n)] for S in self.sets],
                        dtype=np.float64).reshape(len(self.sets), self.g.n)

    def subsets(self):
        """For every j the indices i < j with L_i a proper subset of L_j, and
        dt, dm, c of those pairs."""
        X = self.member()
        Bd = np.array([[S >> v & 1 for v in range(self.g.n)] for S in self.bd],
                      dtype=np.float64).reshape(X.shape)
        T, M = np.array(self.T, dtype=np.float64), np.array(self.M, dtype=np.float64)
        size, Ms = X.sum(1), X @ M
        for j in range(1, len(self.sets)):
            i = np.nonzero((X[:j] @ X[j] == size[:j]) & (size[:j] < size[j]))[0]
            out = X[j] - X[i]
            yield (j, i, (out * (1 - Bd[j]) @ T).astype(np.int64),
                   ((1 - X[i]) * Bd[j] @ M).astype(np.int64),
                   (2 * (Ms[j] - Ms[i]) + self.A[j]).astype(np.int64))


_work_cache = {}


def work(case):
    """Bytes: the table written once, in cells of 16 (32) bits, and the results.
    Flops: three integer operations (budget test, addition, minimum) for every
    relaxation, one (L, L', t) of Algorithm 1's loop with a source cell in its
    row's support; of the memory-indexed table, with a memory in its row."""
    key = repr(sorted((k, v) for k, v in case.items() if k != "name"))
    if key in _work_cache:
        return dict(_work_cache[key])
    g = _graph(case, 0)
    mod = _Model(g, case["mode"])
    X = mod.member().astype(np.float32)
    size = X.sum(1)
    w = np.array(mod.w, dtype=np.float64)
    F, relax = len(mod.sets), 0.0
    cells = float(w.sum())
    B = _budget(case, g)
    width = 4 if min(B, 2 * sum(g.M)) > 65532 else 2
    if case["call"].startswith("dual"):
        w = np.full(F, float(min(B, sum(g.M)) + 1))
        cells, width = float(w.sum()), 4
    for a in range(0, F, 512):
        sub = (X[a:a + 512] @ X.T == size[None, :]) & (size[None, :] < size[a:a + 512, None])
        relax += float((sub @ w).sum())
    tables = case.get("budgets", 1)
    out = cells * width * tables + 13.0 * g.n * tables
    if case["call"] == "table":
        out += 12.0 * F * (sum(g.T) + 1)
    _work_cache[key] = {"bytes": out, "flops": 3.0 * relax * tables}
    return dict(_work_cache[key])


def tolerance(case):
    """Whole numbers throughout: sizes, times, set indices."""
    return "exact"


_BIG = 1 << 60


def _evaluate(mod, chain):
    """seg, cached, Eq. 1, Eq. 2 and M(U_k) of an increasing chain."""
    n = mod.g.n
    seg = np.zeros(n, dtype=np.int32)
    U, prev, peak = 0, 0, 0
    for i, x in enumerate(chain):
        L = mod.sets[x]
        for v in _nodes(L & ~prev):
            seg[v] = i
        peak = max(peak, mod.sum(mod.M, U) + 2 * mod.sum(mod.M, L & ~prev) + mod.A[x])
        U |= mod.bd[x]
        prev = L
    return {"chain": _padded(chain, n), "seg": seg,
            "cached": np.array([bool(U >> v & 1) for v in range(n)], dtype=bool),
            "overhead": mod.sum(mod.T, prev & ~U), "peak": peak, "cache_mem": mod.sum(mod.M, U)}


def _front(row):
    """The row's weak front: cells no larger than every earlier one."""
    least = np.minimum.accumulate(np.concatenate(([_BIG], row[:-1])))
    return np.where(row <= least, row, _BIG)


def exact(case, seed):
    """Algorithm 1 in numpy, 64-bit integers; None where it takes too long, for
    the sweep, and for the schedule of the memory-indexed table (its own tie
    rule)."""
    call, objective = case["call"], case["objective"]
    if call == "sweep" or work(case)["flops"] > 1.5e9:
        return None
    g = _graph(case, seed)
    if g.n > 100 and case["costs"] != "t10":
        return None
    mod = _Model(g, case["mode"])
    F = len(mod.sets)
    if F > 1500:
        return None
    B = _budget(case, g)
    width = sum(g.T) + 1
    opt = [np.full(w, _BIG, dtype=np.int64) for w in mod.w]
    arg = [np.full(w, -1, dtype=np.int32) for w in mod.w]
    opt[0][0] = 0
    for j, src, dt, dm, c in mod.subsets():
        for i, d, a, cc in zip(src.tolist(), dt.tolist(), dm.tolist(), c.tolist()):
            if B < cc:
                continue
            x = opt[i]
            y = np.where(x <= B - cc, x + a, _BIG)
            n = min(len(y), len(opt[j]) - d)
            if n <= 0:
                continue
            o, r = opt[j][d:d + n], arg[j][d:d + n]
            better = y[:n] < o
            o[better] = y[:n][better]
            r[better] = i
        if call == "dominance":
            kept = _front(opt[j])
            arg[j][kept >= _BIG] = -1
            opt[j] = kept
    finite = np.nonzero(opt[-1] < _BIG)[0]
    t = -1 if len(finite) == 0 else int(finite[0] if objective == "tc" else finite[-1])
    out = {"t": t, "m": int(opt[-1][t]) if t >= 0 else -1}
    if call == "table":
        out["table"] = np.full((F, width), -1, dtype=np.int64)
        out["optarg"] = np.full((F, width), -1, dtype=np.int32)
        for j in range(F):
            out["table"][j, :mod.w[j]] = np.where(opt[j] < _BIG, opt[j], -1)
            out["optarg"][j, :mod.w[j]] = arg[j]
        return out
    if t < 0:
        return out
    if call.startswith("dual"):
        out.update(dict.fromkeys(("chain", "seg", "cached", "overhead", "peak", "cache_mem")))
        return out
    steps = {j: dict(zip(src.tolist(), dt.tolist())) for j, src, dt, _, _ in mod.subsets()}
    chain, j, tt = [], F - 1, t
    while j:
        chain.append(j)
        i = int(arg[j][tt])
        tt -= steps[j][i]
        j = i
    out.update(_evaluate(mod, chain[::-1]))
    return out
