"""The work that programs have this library do, as cases to be timed.

A case is one weighted model count, one batch of counts or one burst of
serving requests through the library's public entry points (``wmc_contract``,
``Batch.contract``, ``Server.submit`` / ``drain``).  The formula and the
options of the plan belong to the case; a program plans once, keeps the plan
and its workspace, and comes back with new literal weights: those are what a
seed draws.  Every result is (mantissa, exponent), W = mantissa * 2^exp2, as
the library returns it; counts of plans in scaled FP32 are handed on in
float32, the precision that they are computed to.

Forms of a formula (``form``):

* ``kcnf``    uniform random 3-CNF: the smallest calls, where latency counts
* ``banded``  random 3-CNF whose clauses stay inside a window of variables
* ``lattice`` binary clauses on the edges of a grid plus local ternary ones,
              and (``n_global``) 3-clauses across the whole grid
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2006_15512_amd as W
import wmc_workloads as wl


def listed():
    return [
        # one small formula at a time: every query of an interactive program,
        # an equivalence check or a cell of a parameter sweep
        dict(name="solo_20var_fp64", mode="solo", form="kcnf", n=20, m=85, fseed=2, kind="minfill", tseed=0,
             block=1, precision="fp64"),
        # one formula of middling size: ragged count of variables, FP32
        dict(name="solo_banded123_fp32", mode="solo", form="banded", n=123, m=455, window=20, fseed=0,
             kind="minfill", tseed=0, block=1, precision="fp32"),
        # one structure of the serving set counted alone: long narrow lattice
        dict(name="solo_lattice10x20_fp64", mode="solo", form="lattice", rows=10, cols=20, ternary=0.20, n_global=0,
             fseed=2, kind="minfill", tseed=0, block=1, precision="fp64"),
        # wide lattice swept row by row: matrix-shaped contractions of a
        # 2^24-entry frontier, in both storage precisions
        dict(name="lattice24_sweep_fp64", mode="solo", form="lattice", rows=24, cols=24, ternary=0.10, n_global=0,
             fseed=0, kind="order", tseed=0, block=5, precision="fp64"),
        dict(name="lattice24_sweep_fp32", mode="solo", form="lattice", rows=24, cols=24, ternary=0.10, n_global=0,
             fseed=0, kind="order", tseed=0, block=5, precision="fp32"),
        # the same lattice on the tree that needs no knowledge of it: rank 33
        # sliced to 26, many slices side by side
        dict(name="lattice24_minfill_fp64", mode="solo", form="lattice", rows=24, cols=24, ternary=0.10, n_global=0,
             fseed=0, kind="minfill", tseed=0, block=3, rank_cap=26, slice_group=16, precision="fp64"),
        # the largest formula: banded, 300 variables, rank 29 sliced to 27
        dict(name="banded300_fp64", mode="solo", form="banded", n=300, m=1050, window=37, fseed=0, kind="minfill",
             tseed=5, block=4, rank_cap=27, slice_group=8, precision="fp64"),
        dict(name="banded300_fp32", mode="solo", form="banded", n=300, m=1050, window=37, fseed=0, kind="minfill",
             tseed=5, block=4, rank_cap=27, slice_group=8, precision="fp32"),
        # many independent formulas with new weights each time, replayed
        dict(name="batch512_fp64", mode="batch", count=512, first=0, replay=True, precision="fp64"),
        dict(name="batch512_fp32", mode="batch", count=512, first=0, replay=True, precision="fp32"),
        # weight queries against registered structures: a handful in FP64,
        # and a burst that fills the server's slots in FP32
        dict(name="serve5_fp64", mode="serve", queries=5, qseed=0, slots=16, precision="fp64"),
        dict(name="serve192_fp32", mode="serve", queries=192, qseed=0, slots=128, precision="fp32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    precision = rng.choice(["fp64", "fp32"])
    pick = rng.choice(["kcnf", "banded", "banded", "lattice", "sweep", "sweep", "sliced", "batch", "batch", "serve"])
    fseed = rng.randrange(1000)
    if pick == "kcnf":
        n = rng.randrange(5, 25)
        return dict(mode="solo", form="kcnf", n=n, m=int(round(n * rng.uniform(2.0, 4.25))), fseed=fseed,
                    kind="minfill", tseed=rng.randrange(16), block=rng.choice([1, 1, 2]), precision=precision)
    if pick == "banded":
        n = _log_int(rng, 30, 300)
        return dict(mode="solo", form="banded", n=n, m=int(round(n * rng.uniform(3.0, 4.2))),
                    window=min(n, rng.randrange(8, 29)), fseed=fseed, kind="minfill", tseed=rng.randrange(16),
                    block=rng.randrange(1, 5), precision=precision)
    if pick == "lattice":
        return dict(mode="solo", form="lattice", rows=rng.randrange(4, 14), cols=rng.randrange(5, 25),
                    ternary=round(rng.uniform(0.0, 0.3), 3), n_global=rng.choice([0, 0, 2]), fseed=fseed,
                    kind="minfill", tseed=rng.randrange(16), block=rng.randrange(1, 4), precision=precision)
    if pick == "sweep":
        return dict(mode="solo", form="lattice", rows=rng.randrange(6, 25), cols=rng.randrange(12, 25),
                    ternary=round(rng.uniform(0.0, 0.2), 3), n_global=0, fseed=fseed, kind="order", tseed=0,
                    block=rng.randrange(1, 7), precision=precision)
    if pick == "sliced":
        cols = rng.randrange(12, 19)
        return dict(mode="solo", form="lattice", rows=cols + rng.randrange(0, 5), cols=cols,
                    ternary=round(rng.uniform(0.0, 0.2), 3), n_global=0, fseed=fseed, kind="minfill",
                    tseed=rng.randrange(16), block=rng.randrange(1, 4), rank_cap=cols + rng.randrange(3, 5),
                    slice_group=rng.choice([1, 4, 16]), precision=precision)
    if pick == "batch":
        count = _log_int(rng, 3, 512)
        return dict(mode="batch", count=count, first=rng.randrange(0, 513 - count), replay=rng.random() < 0.6,
                    precision=precision)
    return dict(mode="serve", queries=_log_int(rng, 1, 300), qseed=fseed, slots=rng.choice([8, 32, 128]),
                precision=precision)


# --------------------------------------------------------------------------
# formulas and plans
# --------------------------------------------------------------------------
def _formula(case):
    if case["form"] == "kcnf":
        return wl.random_kcnf(case["n"], case["m"], seed=case["fseed"])
    if case["form"] == "banded":
        return wl.banded_3cnf(case["n"], case["m"], case["window"], seed=case["fseed"])
    return wl.grid_cnf(case["rows"], case["cols"], case["ternary"], seed=case["fseed"], n_global=case["n_global"])


def _plan(case, f):
    order = wl.row_major_order(case["rows"], case["cols"]) if case["kind"] == "order" else None
    return W.Plan(W.Network.from_formula(f), kind=case["kind"], seed=case["tseed"], order=order, block=case["block"],
                  rank_cap=case.get("rank_cap", 0), slice_group=case.get("slice_group", 1),
                  precision=case["precision"])


def _weights(rng, n, lo=0.1, hi=0.9):
    """Literal weights {1 - w, w}, w ~ U(lo, hi), as (n, 2)."""
    return wl.uniform_weights(rng, n, lo, hi)


def _solo_weights(case, f, seed):
    lo, hi = (0.05, 0.95) if case["form"] == "banded" else (0.1, 0.9)
    return _weights(np.random.default_rng(seed), f.n, lo, hi)


_instance = functools.lru_cache(maxsize=None)(wl.batch_instance)
_structure = functools.lru_cache(maxsize=None)(wl.serve_structure)


def _batch_formulas(case):
    return [_instance(i) for i in range(case["first"], case["first"] + case["count"])]


def _batch_weights(formulas, seed):
    rng = np.random.default_rng(seed)
    return [_weights(rng, f.n) for f in formulas]


def _queries(case, seed):
    """(structure of each query, its weights): which structures are asked
    belongs to the case, the weights to the seed."""
    which = np.random.default_rng(case["qseed"]).integers(0, len(wl.SERVE_STRUCTURES), size=case["queries"])
    rng = np.random.default_rng(seed)
    return [int(s) for s in which], [_weights(rng, 200) for _ in which]


# --------------------------------------------------------------------------
# the measured interface
# --------------------------------------------------------------------------
def prepare(case, seed):
    real = np.float64 if case["precision"] == "fp64" else np.float32
    state = dict(mode=case["mode"], real=real)
    if case["mode"] == "solo":
        f = _formula(case)
        state["plan"] = _plan(case, f)
        state["ws"] = W.workspace(state["plan"])
        state["weights"] = _solo_weights(case, f, seed)
    elif case["mode"] == "batch":
        fs = _batch_formulas(case)
        state["batch"] = W.Batch([W.Plan(W.Network.from_formula(f), kind="minfill", seed=0,
                                         precision=case["precision"]) for f in fs])
        state["ws"] = state["batch"].workspace()
        state["weights"] = np.concatenate([w.reshape(-1) for w in _batch_weights(fs, seed)])
        state["flags"] = W.BATCH_GRAPH | W.BATCH_RESIDENT if case["replay"] else 0
    else:
        srv = W.Server(precision=case["precision"], max_slots=case["slots"], hbm_budget_bytes=6 << 30,
                       buffer_bytes=7 << 30)
        for s in range(len(wl.SERVE_STRUCTURES)):
            srv.register(W.Plan(W.Network.from_formula(_structure(s)), kind="minfill", seed=0,
                                precision=case["precision"]))
        state["server"] = srv
        state["which"], state["weights"] = _queries(case, seed)
    return state


def run(state):
    if state["mode"] == "solo":
        values = [W.wmc_contract(state["plan"], state["weights"], state["ws"])]
    elif state["mode"] == "batch":
        values = state["batch"].contract(state["weights"], ws=state["ws"], flags=state["flags"])
    else:
        srv = state["server"]
        for i, (s, w) in enumerate(zip(state["which"], state["weights"])):
            srv.submit(s, w, i)
        done = srv.drain()
        values = [r.value for r in sorted(done, key=lambda r: r.request_id)]
    return dict(mantissa=np.array([v.mantissa for v in values], dtype=state["real"]),
                exp2=np.array([v.exp2 for v in values], dtype=np.int64))


def _plan_work(plans):
    stats = [p.stats() for p in plans]
    return dict(bytes=sum(s["bytes_per_slice"] * s["n_slices"] for s in stats),
                flops=sum(s["flops_per_slice"] * s["n_slices"] for s in stats))


def work(case):
    """Every tensor of the contraction tree written once and read once, and
    the multiplications and additions of its pairwise contractions."""
    if case["mode"] == "solo":
        return _plan_work([_plan(case, _formula(case))])
    if case["mode"] == "batch":
        return _plan_work([W.Plan(W.Network.from_formula(f), kind="minfill", seed=0, precision=case["precision"])
                           for f in _batch_formulas(case)])
    plans = [W.Plan(W.Network.from_formula(_structure(s)), kind="minfill", seed=0,
                    precision=case["precision"]) for s in range(len(wl.SERVE_STRUCTURES))]
    return _plan_work([plans[s] for s in _queries(case, 0)[0]])


# --------------------------------------------------------------------------
# the same counts in 64 bits, by plain variable elimination in torch
# --------------------------------------------------------------------------
def _min_fill(n, clauses):
    """Elimination order (0-based) of least fill; neighbourhoods as bit sets."""
    nb = [0] * n
    for c in clauses:
        mask = 0
        for l in c:
            mask |= 1 << (abs(l) - 1)
        for l in c:
            nb[abs(l) - 1] |= mask
    nb = [m & ~(1 << v) for v, m in enumerate(nb)]
    left, order = set(range(n)), []

    def bits(m):
        while m:
            low = m & -m
            yield low.bit_length() - 1
            m ^= low

    cost = {}
    while left:
        best = None
        for v in left:
            if v not in cost:
                cost[v] = sum(bin(nb[v] & ~nb[u] & ~(1 << u)).count("1") for u in bits(nb[v]))
            key = (cost[v], bin(nb[v]).count("1"), v)
            if best is None or key < best:
                best = key
        v = best[2]
        around = nb[v]
        stale = around
        for u in bits(around):
            nb[u] = (nb[u] | around) & ~(1 << u) & ~(1 << v)
            stale |= nb[u]
        for u in bits(stale):
            cost.pop(u, None)
        cost.pop(v, None)
        left.discard(v)
        order.append(v)
    return order


def _times(va, a, vb, b):
    """Product of two tables over ascending scopes, as one table over their
    union (the first variable of a scope is the most significant bit)."""
    vs = sorted(set(va) | set(vb))
    sa, sb = set(va), set(vb)
    dims, last = [], None
    for v in vs:
        k = (v in sa, v in sb)
        if k == last:
            dims[-1][0] *= 2
        else:
            dims.append([2, k])
            last = k
    da = [d if k[0] else 1 for d, k in dims]
    db = [d if k[1] else 1 for d, k in dims]
    full = [d for d, _ in dims]
    a, b = a.reshape(da), b.reshape(db)
    if len(full) <= 12:
        return vs, (a * b).reshape(-1)
    out = torch.empty(full, dtype=a.dtype, device=a.device)  # too many axes for one elementwise kernel

    def part(o, x, y, axes):
        if axes <= 12:
            torch.mul(x, y, out=o)
            return
        for i in range(o.shape[0]):
            part(o[i], x[i if x.shape[0] > 1 else 0], y[i if y.shape[0] > 1 else 0], axes - 1)

    part(out, a, b, len(full))
    return vs, out.reshape(-1)


def _count(n, clauses, weights, order, device):
    """W of one formula as a one-entry tensor; order is 0-based."""
    at = [0] * n
    for p, v in enumerate(order):
        at[v] = p
    table = {}
    buckets = [[] for _ in range(n)]
    w = torch.from_numpy(np.ascontiguousarray(np.asarray(weights, dtype=np.float64)[np.asarray(order)])).to(device)
    for p in range(n):
        buckets[p].append(([p], w[p]))
    for c in clauses:
        vs = sorted({at[abs(l) - 1] for l in c})
        false = 0
        for l in c:
            false |= (1 if l < 0 else 0) << (len(vs) - 1 - vs.index(at[abs(l) - 1]))
        key = (len(vs), false)
        if key not in table:
            t = torch.ones(1 << len(vs), dtype=torch.float64, device=device)
            t[false] = 0.0
            table[key] = t
        buckets[vs[0]].append((vs, table[key]))
    out = torch.ones(1, dtype=torch.float64, device=device)
    for p in range(n):
        fs = sorted(buckets[p], key=lambda f: len(f[0]))
        buckets[p] = None
        vs, t = fs[0]
        for ws, u in fs[1:]:
            vs, t = _times(vs, t, ws, u)
        t = t.reshape(2, -1)
        t = t[0] + t[1]
        if len(vs) > 1:
            buckets[vs[1]].append((vs[1:], t))
        else:
            out = out * t
    return out


def exact(case, seed):
    device = "cuda:0" if torch.cuda.is_available() else "cpu"
    if case["mode"] == "solo":
        f = _formula(case)
        if case["form"] == "lattice" and case["kind"] == "order":
            order = list(range(f.n))
        elif case["form"] == "lattice" and case["n_global"] == 0:  # along the shorter side
            r, c = case["rows"], case["cols"]
            order = [i * c + j for j in range(c) for i in range(r)] if r < c else list(range(f.n))
        else:
            order = _min_fill(f.n, f.clauses)
        found = [_count(f.n, f.clauses, _solo_weights(case, f, seed), order, device)]
    elif case["mode"] == "batch":
        fs = _batch_formulas(case)
        found = [_count(f.n, f.clauses, w, range(f.n), device) for f, w in zip(fs, _batch_weights(fs, seed))]
    else:
        which, weights = _queries(case, seed)
        fs = {s: _structure(s) for s in set(which)}
        orders = {s: _min_fill(f.n, f.clauses) for s, f in fs.items()}
        found = [_count(fs[s].n, fs[s].clauses, w, orders[s], device) for s, w in zip(which, weights)]
    m, e = np.frexp(torch.cat(found).cpu().numpy())
    return dict(mantissa=m, exp2=np.where(m == 0.0, 0, e).astype(np.int64))
