"""The work that a user of the solver has it do, as cases that can be timed
and whose results can be compared.

Every case goes through the public Python entry points (Context.load / solve /
solve_batch / root / lns, Policy.train_step / grad / forward) with the knobs a
user would set.  Instances come from the repository's seeded generators; the
seed given to prepare() picks them.  What run() returns does not depend on the
schedule of the parallel search: solution sets in sorted order, exact counts,
and the node and failure counts of exhausted trees (a find-first launch under
a node budget returns those of the instances it proved infeasible; which
solution the others report is the schedule's choice).
"""
import itertools
import math

import numpy as np
import torch

import cspgen
from paper_1909_09213_amd import cubics as cb
from paper_1909_09213_amd import learn

F, H = learn.F, learn.H
_contexts = {}


def _ctx():
    """One context per process, as a user's program keeps it."""
    if "ctx" not in _contexts:
        _contexts["ctx"] = cb.Context(0)
    return _contexts["ctx"]


def listed():
    return [
        # the smallest search: all solutions of 8-queens with blocked squares
        {"name": "queens8_all", "kind": "queens", "n": 8, "blocked": 4, "all": True},
        # one puzzle counted exhaustively, arithmetic constraints
        {"name": "queens13_count", "kind": "queens", "n": 13, "blocked": 8, "all": False},
        # one random binary CSP counted exhaustively (n=40, d=16, 195 tables)
        {"name": "rb40_count", "kind": "rb", "n": 40, "d": 16, "dens_pm": 250, "tight_pm": 380, "two_way": False},
        # the same family past its solutions: a small tree, all latency
        {"name": "rb40_sparse", "kind": "rb", "n": 40, "d": 16, "dens_pm": 250, "tight_pm": 400, "two_way": False},
        # the batched sweep: find-first over n 20..120, d 8..64 with a node budget
        {"name": "sweep_first", "kind": "sweep", "batch": 320, "budget": 20000, "active": 8},
        # labels of the learned ordering: many sub-CSPs counted in one launch
        {"name": "label_batch", "kind": "labels", "batch": 768, "n_hi": 24, "learned": False},
        # held-out instances counted under a learned variable order
        {"name": "learned_batch", "kind": "labels", "batch": 192, "n_hi": 24, "learned": True},
        # first solutions under a learned value order, one worker per instance
        {"name": "value_order_first", "kind": "first", "batch": 512, "n_hi": 28, "value_policy": True},
        # all-different + linear instances (plain, GAC, group-bounded) in one batch
        {"name": "global_batch", "kind": "twins", "batch": 48, "n": 7, "d": 8},
        # a slice of the n=200, d=256 all-different + linear family (8 words per domain)
        {"name": "global_wide", "kind": "wide", "n": 200, "d": 256, "free": 3, "vals": 64, "split": 4096},
        # the root fixpoint of the sweep's largest instance shape
        {"name": "root_n120_d64", "kind": "root", "family": "rb", "n": 120, "d": 64},
        # one full-batch training step of the policy network (records of a 20,000-instance run)
        {"name": "train_135797", "kind": "mlp", "op": "train", "rows": 135797},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tightness(n, d, dens_pm, bits):
    """Per-mille tightness at which an n-variable random binary CSP has about
    2**bits solutions on average."""
    m = max(1, (dens_pm * n * (n - 1) // 2 + 500) // 1000)
    keep = 2.0 ** (-(n * math.log2(d) - bits) / m)
    return int(min(900, max(50, round(1000 * (1 - keep)))))


def draw(rng):
    kind = rng.choice(["queens", "queens", "rb", "rb", "sweep", "labels", "labels", "first", "twins", "wide",
                       "root", "root", "mlp", "mlp", "lns"])
    if kind == "queens":
        n = rng.randint(6, 13)
        return {"kind": kind, "n": n, "blocked": rng.randint(n // 2, n), "all": n <= 9 and rng.random() < 0.5}
    if kind == "rb":
        n, d, dens = rng.randint(16, 40), rng.randint(6, 24), rng.randint(250, 450)
        return {"kind": kind, "n": n, "d": d, "dens_pm": dens,
                "tight_pm": _tightness(n, d, dens, rng.uniform(8, 22)), "two_way": rng.random() < 0.2}
    if kind == "sweep":
        return {"kind": kind, "batch": _log_int(rng, 64, 256), "budget": _log_int(rng, 1000, 20000),
                "active": rng.choice([0, 4, 8])}
    if kind == "labels":
        learned = rng.random() < 0.4
        return {"kind": kind, "batch": _log_int(rng, 24, 180 if learned else 700), "n_hi": rng.randint(15, 24),
                "learned": learned}
    if kind == "first":
        return {"kind": kind, "batch": _log_int(rng, 32, 500), "n_hi": rng.randint(18, 28),
                "value_policy": rng.random() < 0.6}
    if kind == "twins":
        return {"kind": kind, "batch": _log_int(rng, 6, 48), "n": rng.randint(5, 7), "d": rng.randint(5, 8)}
    if kind == "wide":
        return {"kind": kind, "n": rng.randint(40, 200), "d": rng.randint(33, 256), "free": rng.randint(2, 3),
                "vals": rng.randint(12, 32), "split": rng.choice([0, 512, 4096])}
    if kind == "root":
        return {"kind": kind, "family": rng.choice(["rb", "rb", "tree", "global", "gac"]),
                "n": _log_int(rng, 20, 120), "d": _log_int(rng, 8, 64)}
    if kind == "mlp":
        return {"kind": kind, "op": rng.choice(["train", "grad", "forward"]), "rows": _log_int(rng, 100, 1_000_000)}
    return {"kind": "lns", "n": rng.randint(10, 18), "d": rng.randint(5, 8), "copies": _log_int(rng, 16, 128)}


# ---------------------------------------------------------------- instances

def _blocked_queens(case, r):
    """n-queens with `blocked` squares that hold no queen."""
    n = case["n"]
    q = cspgen.queens(n)
    init = q.full_init()
    for s in r.choice(n * n, size=case["blocked"], replace=False):
        init[s // n, 0] &= ~np.uint32(1 << (s % n))
    return q.with_init(init)


def _small_csps(case, r, count, bits_lo, bits_hi):
    """Random binary CSPs at the sizes of the learned-branching workload, some
    with one or two variables fixed (the children of a search node)."""
    out = []
    for _ in range(count):
        n, d = int(r.integers(12, case["n_hi"] + 1)), int(r.integers(6, 13))
        dens = int(r.integers(350, 551))
        tight = _tightness(n, d, dens, r.uniform(bits_lo, bits_hi))
        x = cspgen.rb(int(r.integers(1 << 30)), n=n, d=d, dens_pm=dens, tight_pm=tight, base=901)
        k = int(r.integers(0, 3))
        out.append(x.fix({int(i): int(r.integers(d)) for i in r.choice(n, size=k, replace=False)}) if k else x)
    return out


def _wide_slice(case, r):
    """A slice of an all-different + linear instance: every variable fixed to
    a value of one assignment that satisfies all constraints, except `free`
    ones that choose among `vals` values."""
    n, d = case["n"], case["d"]
    k = max(2, min(20, n // 10, d // 2))
    g = cspgen.global_family(int(r.integers(1 << 30)), n=n, lo=0, d=d, n_ad=max(1, n // 20), k_ad=k,
                             n_lin=max(1, 3 * n // 20), base=902)
    hi = max(k + 1, int(0.8 * d))
    while True:
        point = r.permutation(n)[:n] % hi if n > hi else r.permutation(hi)[:n]
        ok = True
        for c in range(g.m):
            v = point[g.scope(c)]
            if g.type[c] == cspgen.LINEAR_LE:
                ok = ok and int((np.asarray(g.par(c)[1:]) * v).sum()) <= int(g.par(c)[0])
            else:
                ok = ok and len(set(v.tolist())) == len(v)
        if ok:
            break
    init = np.zeros((n, g.W), dtype=np.uint32)
    init[np.arange(n), point // 32] = np.uint32(1) << (point % 32).astype(np.uint32)
    for i in r.choice(n, size=case["free"], replace=False):
        init[i] = 0
        for v in r.choice(d, size=min(d, case["vals"]), replace=False):
            init[i, v // 32] |= np.uint32(1) << np.uint32(v % 32)
    return g.with_init(init)


def _root_instance(case, r):
    n, d, s = case["n"], case["d"], int(r.integers(1 << 30))
    if case["family"] == "tree":
        return cspgen.tree(s, n, d, 600, base=903)
    if case["family"] == "rb":
        x = cspgen.rb(s, n=n, d=d, dens_pm=300, tight_pm=350, base=903)
    else:
        k = max(2, min(d // 2, n // 4))
        x = cspgen.global_family(s, n=n, lo=0, d=d, n_ad=max(1, n // 10), k_ad=k, n_lin=n // 7, b_pm=300, base=903)
        x = x.with_gac() if case["family"] == "gac" else x
    # a node of a search: one variable assigned, a few others down to five to
    # seven values
    init = x.full_init()
    for q, i in enumerate(r.choice(n, size=max(2, n // 10), replace=False)):
        init[i] = 0
        for v in r.choice(d, size=min(d, int(r.integers(5, 8))) if q else 1, replace=False):
            init[i, v // 32] |= np.uint32(1) << np.uint32(v % 32)
    return x.with_init(init)


def _theta(r):
    """Parameters of a branching or value network; the failure-count feature
    has zero weight, as training on sampled nodes leaves it."""
    th = np.zeros(cb.Policy.NP, dtype=np.float32)
    w1 = r.normal(0, math.sqrt(2.0 / F), (H, F))
    w1[:, F - 1] = 0
    th[:H * F] = w1.reshape(-1)
    th[H * F:H * F + H] = 0.01
    th[H * F + H:H * F + 2 * H] = r.normal(0, math.sqrt(1.0 / H), H)
    return th


def _records(rows, seed):
    """Trace records [rows, 8]: five features in [0, 1], group columns, and a
    centred label in column 7."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rec = torch.rand(rows, 8, device="cuda", generator=g)
    rec[:, 7] = 2 * torch.randn(rows, device="cuda", generator=g)
    return rec


# ------------------------------------------------------------------- cases

def prepare(case, seed):
    ctx, r, kind = _ctx(), np.random.default_rng(seed), case["kind"]
    s = {"kind": kind, "ctx": ctx}
    if kind == "queens":
        s["prob"] = ctx.load(_blocked_queens(case, r))
        s["kw"] = ({"mode": cb.MODE_ALL, "sol_capacity": 1024} if case["all"] else {"mode": cb.MODE_COUNT})
    elif kind == "rb":
        inst = cspgen.rb(int(r.integers(1 << 30)), n=case["n"], d=case["d"], dens_pm=case["dens_pm"],
                         tight_pm=case["tight_pm"], base=904)
        s["prob"], s["kw"] = ctx.load(inst), {"mode": cb.MODE_COUNT, "two_way": case["two_way"]}
    elif kind == "wide":
        s["prob"] = ctx.load(_wide_slice(case, r))
        s["kw"] = {"mode": cb.MODE_COUNT, "split_target": case["split"]}
    elif kind == "sweep":
        first = int(r.integers(1 << 40))
        s["probs"] = [ctx.load(cspgen.rb_sweep(first + i)) for i in range(case["batch"])]
        s["kw"] = {"mode": cb.MODE_FIRST, "max_nodes": case["budget"], "layout": cb.LAYOUT_LANE,
                   "active_per_xcd": case["active"],
                   "sol_out": torch.zeros((case["batch"], 128), dtype=torch.int32, device="cuda")}
    elif kind == "labels":
        s["probs"] = [ctx.load(x) for x in _small_csps(case, r, case["batch"], 4, 15)]
        s["kw"] = {"mode": cb.MODE_COUNT}
        if case["learned"]:
            s["policy"] = cb.Policy(ctx, _theta(r))
            s["kw"].update(branching=cb.BRANCH_LEARNED, policy=s["policy"], layout=cb.LAYOUT_LANE)
    elif kind == "first":
        s["probs"] = [ctx.load(x) for x in _small_csps(case, r, case["batch"], 10, 24)]
        s["sol"] = torch.zeros((case["batch"], 32), dtype=torch.int32, device="cuda")
        s["kw"] = {"mode": cb.MODE_FIRST, "donate": False, "layout": cb.LAYOUT_LANE, "sol_out": s["sol"]}
        if case["value_policy"]:
            s["policy"] = cb.Policy(ctx, _theta(r))
            s["kw"]["value_policy"] = s["policy"]
    elif kind == "twins":
        make = (lambda x: x, lambda x: x.with_gac(), lambda x: x.with_linear_ad())
        s["probs"] = [ctx.load(make[i % 3](cspgen.global_family(
            int(r.integers(1 << 30)), n=case["n"], lo=0, d=case["d"], n_ad=2, k_ad=(case["n"] + 1) // 2, n_lin=3,
            base=905))) for i in range(case["batch"])]
        s["kw"] = {"mode": cb.MODE_COUNT}
    elif kind == "root":
        s["prob"] = ctx.load(_root_instance(case, r))
    elif kind == "lns":
        s["inst"] = cspgen.rb(int(r.integers(1 << 30)), n=case["n"], d=case["d"], dens_pm=300,
                              tight_pm=_tightness(case["n"], case["d"], 300, 12), base=906)
        s["obj"], s["copies"] = r.integers(1, 10, case["n"]), case["copies"]
    else:
        s["op"], s["rec"] = case["op"], _records(case["rows"], seed)
        s["policy"] = cb.Policy(ctx, _theta(r))
    return s


def _counts(res):
    return np.array([[r.count, r.nodes, r.fails] for r in res], dtype=np.int64)


def _in_order(solutions, rows):
    """The solution set in lexicographic order, padded with zero rows (the
    search stores solutions in the order it meets them)."""
    out = np.zeros((rows, solutions.shape[1]), dtype=np.int64)
    out[:len(solutions)] = solutions[np.lexsort(solutions.T[::-1])]
    return out


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind in ("queens", "rb", "wide"):
        r = ctx.solve(state["prob"], **state["kw"])
        out = {"counts": _counts([r])}
        if r.solutions is not None:
            out["solutions"] = _in_order(r.solutions, state["kw"]["sol_capacity"])
        return out
    if kind == "sweep":
        res = ctx.solve_batch(state["probs"], **state["kw"])
        return np.array([[r.nodes, r.fails] if r.verdict == "UNSAT" else [0, 0] for r in res], dtype=np.int64)
    if kind in ("labels", "twins"):
        return _counts(ctx.solve_batch(state["probs"], **state["kw"]))
    if kind == "first":
        return {"counts": _counts(ctx.solve_batch(state["probs"], **state["kw"])), "solutions": state["sol"]}
    if kind == "root":
        failed, dom = ctx.root(state["prob"])
        return {"failed": failed, "domains": np.where(failed, 0, dom).astype(np.int64)}
    if kind == "lns":
        r = ctx.lns(state["inst"], state["obj"], neighborhoods=state["copies"], relax_pm=300, max_nodes=1_000_000)
        return {"objective": r["objective"] if r["found"] else -1, "optimal": r["optimal"]}
    pol = state["policy"]
    if state["op"] == "forward":
        return pol.forward(state["rec"])
    if state["op"] == "grad":
        return pol.grad(state["rec"])
    loss = pol.train_step(state["rec"], 1e-2, 1)
    return {"theta": pol.get(), "loss": loss}


def _table_words(n, d, dens_pm):
    return (dens_pm * n * (n - 1) / 2000) * d * ((d + 31) // 32)


def work(case):
    """Bytes of the inputs and outputs: the constraint tables, domains and
    coefficients of every instance, or the records."""
    kind = case["kind"]
    if kind == "queens":
        n = case["n"]
        return {"bytes": 12.0 * n * (n - 1) / 2 + 12.0 * n + 24, "flops": 0.0}
    if kind == "rb":
        return {"bytes": 4.0 * (_table_words(case["n"], case["d"], case["dens_pm"]) + 3 * case["n"]) + 24, "flops": 0.0}
    if kind == "sweep":
        return {"bytes": case["batch"] * (4.0 * _table_words(70, 36, 200) + 4.0 * 70), "flops": 0.0}
    if kind in ("labels", "first"):
        n = (12 + case["n_hi"]) // 2
        return {"bytes": case["batch"] * (4.0 * _table_words(n, 9, 450) + 16.0 * n + 24), "flops": 0.0}
    if kind == "twins":
        return {"bytes": case["batch"] * (4.0 * 6 * case["n"] + 8.0 * 3 * case["n"] + 24), "flops": 0.0}
    if kind == "wide":
        n = case["n"]
        return {"bytes": 4.0 * n * ((case["d"] + 31) // 32) + 12.0 * n * max(1, 3 * n // 20) + 24, "flops": 0.0}
    if kind == "root":
        n, w = case["n"], (case["d"] + 31) // 32
        tables = {"rb": _table_words(n, case["d"], 300), "tree": n * case["d"] * w}.get(case["family"], 3.0 * n * (n // 7))
        return {"bytes": 4.0 * (tables + 2 * n * w), "flops": 0.0}
    if kind == "lns":
        return {"bytes": 4.0 * (_table_words(case["n"], case["d"], 300) + 4 * case["n"]), "flops": 0.0}
    per_row = 2.0 * H * F + 2 * H
    return {"bytes": 4.0 * case["rows"] * 6 + 4 * 449, "flops": case["rows"] * per_row * (1 if case["op"] == "forward" else 3)}


# ------------------------------------------------------------------- exact

def _bf16(x):
    """The rounding the network's definition applies to inputs, weights and
    activations: nearest bf16, ties to even."""
    return x.to(torch.float32).to(torch.bfloat16).double()


def _network(theta, rec, op):
    th = torch.as_tensor(theta, device=rec.device).double()
    W1, b1 = _bf16(th[:H * F]).reshape(H, F), th[H * F:H * F + H]
    w2, b2 = _bf16(th[H * F + H:H * F + 2 * H]), th[-1]
    x, t = _bf16(rec[:, :F]), rec[:, 7].double()
    pre = x @ W1.T + b1
    act = _bf16(pre.clamp_min(0))
    y = act @ w2 + b2
    if op == "forward":
        return y
    e = y - t
    dy = 2 * e / len(t)
    dpre = torch.where(pre > 0, dy[:, None] * w2[None, :], 0.0)
    grad = torch.cat([(dpre.T @ x).reshape(-1), dpre.sum(0), dy @ act, dy.sum().reshape(1)])
    return grad, (e * e).mean().reshape(1)


def _arc_consistent(inst):
    """Root fixpoint of a CSP of binary tables: (failed, [n, W] bit rows)."""
    d = inst.dsize
    bits = inst.full_init() if inst.init is None else inst.init
    none = np.zeros((inst.n, inst.W), dtype=np.int64)
    dom = [np.array([(int(bits[i, v // 32]) >> (v % 32)) & 1 for v in range(d[i])], dtype=bool) for i in range(inst.n)]
    arcs = []
    for c in range(inst.m):
        i, j = (int(v) for v in inst.scope(c))
        w = inst.tab(c).reshape(d[i], -1)
        ok = np.array([[(int(w[a, b // 32]) >> (b % 32)) & 1 for b in range(d[j])] for a in range(d[i])], dtype=bool) \
            if d[i] * d[j] < 64 else np.unpackbits(
                np.ascontiguousarray(w).view(np.uint8).reshape(d[i], -1), axis=1, bitorder="little")[:, :d[j]].astype(bool)
        arcs += [(i, j, ok), (j, i, ok.T)]
    changed = set(range(inst.n))
    while changed:
        now = set()
        for i, j, ok in arcs:
            if j in changed:
                keep = dom[i] & ok[:, dom[j]].any(axis=1)
                if (keep != dom[i]).any():
                    dom[i] = keep
                    now.add(i)
                    if not keep.any():
                        return True, none
        changed = now
    if any(not v.any() for v in dom):
        return True, none
    out = np.zeros((inst.n, inst.W), dtype=np.int64)
    for i, v in enumerate(dom):
        for a in np.flatnonzero(v):
            out[i, a // 32] |= 1 << (a % 32)
    return False, out


def exact(case, seed):
    kind, r = case["kind"], np.random.default_rng(seed)
    if kind == "mlp":
        rec, th = _records(case["rows"], seed), _theta(r)
        if case["op"] != "train":
            return _network(th, rec, case["op"])
        grad, loss = _network(th, rec, "grad")
        # Adam's first step from zero moments
        step = (1e-2 * grad / (grad.abs() + 1e-8)).cpu().numpy()
        return {"theta": th.astype(np.float64) - step, "loss": float(loss[0])}
    if kind == "root" and case["family"] in ("rb", "tree"):
        failed, dom = _arc_consistent(_root_instance(case, r))
        return {"failed": failed, "domains": dom}
    if kind == "queens" and case["n"] <= 8:
        n = case["n"]
        init = _blocked_queens(case, r).init
        sols = [p for p in itertools.permutations(range(n))
                if all((int(init[i, 0]) >> p[i]) & 1 for i in range(n))
                and all(abs(p[i] - p[j]) != i - j for i in range(n) for j in range(i))]
        out = {"counts": None}
        if case["all"]:
            out["solutions"] = _in_order(np.array(sols, dtype=np.int64).reshape(-1, n) + 1, 1024)
        return out
    return None
