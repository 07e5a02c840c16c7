"""The range of a fused program's chains: their words replayed on the CPU with
the power of two they are stored with and the range bits they report, and on
the device the calls that such a report sends to the launch list."""
import math
from fractions import Fraction

import numpy as np
import pytest

import oracle
import paper_2006_15512_amd as W
import plan_emulator as pe
import wmc_workloads as wl
from plan_emulator import _pext, _sexp
from test_chain import (BITS, CH_C, CH_F, CH_FCOPY, CH_OUT, CH_SRC, CH_TC, CH_TF, CH_TILE_BITS, CH_TILES, CH_WORDS, CH_X,
                        CS_BIT, CS_BIT_O, CS_DST, CS_G, CS_PO, CS_PS, CS_QG, CS_QO, CS_SRC, CS_TBITS, CS_TG, CS_WORDS,
                        CS_X, CX_BITS, CX_LDS, CX_LIST, CX_LOW, _deposit, parse, same, tolerance)

CS_LIFT = 7
TINY = 0.5  # an intermediate whose largest entry is nonzero and below is out of range


def ranged(plan, w, eta=0):
    """(mantissa, exponent, flagged) of a plan's fused program for slice eta,
    as the kernels compute it: every tensor of a chain stored 2^lift larger,
    and whether one of its intermediates left the range."""
    prog, info = parse(plan)
    store = np.float64 if plan.precision == "fp64" else np.float32
    arena = np.full(info["arena_elems"], np.nan, dtype=store)
    mx, ex = np.zeros(info["n_tensors"]), np.zeros(info["n_tensors"], dtype=np.int64)
    off = prog["off"]
    for d in prog["leaves"]:
        e = np.arange(1 << int(d["rank"]))
        bit = lambda p: (e >> p) & 1 if p >= 0 else np.full(len(e), (eta >> (-p - 1)) & 1)
        if d["kind"] == 0:
            a = np.zeros(len(e), dtype=np.int64)
            for q in range(int(d["k"])):
                a |= bit(int(d["pos"][q])) << q
            v = np.where((a != int(d["falsify"])) | bool(d["taut"]), 1.0, 0.0)
        else:
            w0, w1 = w[2 * int(d["var"])], w[2 * int(d["var"]) + 1]
            top = max(abs(w0), abs(w1)) if d["kind"] == 1 else abs(w0 + w1)
            v = np.where(bit(int(d["pos"][0])), w1, w0) if d["kind"] == 1 else np.array([w0 + w1])
            s = math.frexp(float(top))[1]
            v, ex[int(d["tensor"])] = np.ldexp(v, -s), s
        s = v.astype(store)
        arena[int(d["out"]): int(d["out"]) + len(e)] = s
        mx[int(d["tensor"])] = np.max(np.abs(s.astype(np.float64)))
    flagged = False
    for typ, nf, nc, cf, cc, _, _, _ in prog["launches"]:
        assert typ != 2, "matrix nodes are not replayed here"
        done = []
        for d in prog["nodes"][nf: nf + nc]:
            r = np.arange(1 << int(d["rc"]), dtype=np.uint64)
            nk = int(d["nk"])
            k = np.arange(1 << nk)
            A = arena[int(d["a"]) + (_pext(r, d["ra"], int(d["nra"])).astype(np.int64)[:, None] << nk | k)]
            B = arena[int(d["b"]) + (_pext(r, d["rb"], int(d["nrb"])).astype(np.int64)[:, None] << nk | k)]
            sh = _sexp(mx[int(d["ta"])]) + _sexp(mx[int(d["tb"])])
            done.append((int(d["c"]), np.ldexp((A.astype(np.float64) * B).sum(1), -sh).astype(store), int(d["tc"]),
                         ex[int(d["ta"])] + ex[int(d["tb"])] + sh))
        for desc in prog["chains"][cf: cf + cc]:
            c = prog["words"][desc:].astype(np.int64)
            L, ob, n = int(c[0]), int(c[CH_TILE_BITS]), CS_WORDS[int(typ)]
            tiles = c[int(c[CH_TILES]):]
            st = [c[CH_WORDS + i * n: CH_WORDS + (i + 1) * n] for i in range(L)]
            base = lambda x: int(x[0]) + (int(x[1]) << 32)
            lift, shift = int(st[0][CS_LIFT]), [-_sexp(mx[int(s[CS_TG])]) for s in st]
            shift[0] += lift - _sexp(mx[int(c[CH_TF])])
            e_total = ex[int(c[CH_TF])] + sum(ex[int(s[CS_TG])] for s in st) - sum(shift)
            result = np.full(1 << len(plan.tensor(int(c[CH_TC]))[2]), np.nan, dtype=store)
            maps = []
            for i, s in enumerate(st):
                np_, nq, tb = (int(s[0]) >> 8) & 255, int(s[0]) >> 16, int(s[CS_TBITS])
                outs = s[CS_BIT_O:] if typ == 3 else c[CH_OUT:] if i + 1 == L else 1 << np.arange(16)
                if typ == 0:
                    memory = i == 0 and not c[CH_FCOPY]
                    bits = [(int(c[CH_SRC + b]) if memory else int(s[CS_BIT + b]) & 0xFFFF, int(s[CS_BIT + b]) >> 16,
                             int(outs[b])) for b in range(tb)]
                else:
                    bits = [(int(s[CS_BIT + b]), int(s[CS_BIT + BITS + b]), int(outs[b])) for b in range(tb)]
                    bits += [(int(s[CS_PS + q]), 0, int(s[CS_PO + q])) for q in range(np_)]
                    bits += [(0, int(s[CS_QG + q]), int(s[CS_QO + q])) for q in range(nq)]
                e = np.arange(1 << len(bits))
                maps.append([_deposit(e, [x[j] for x in bits]) for j in range(3)])
            largest = [0.0] * L
            for t in np.array_split(np.arange(1 << ob), max(1, (1 << ob) // 32)):
                at = lambda q: _deposit(t, tiles[q * ob: (q + 1) * ob])
                src_t, out_t = base(c[CH_F:]) + at(0), base(c[CH_C:]) + at(1)
                lds = np.full((len(t), 65536 // np.dtype(store).itemsize), np.nan, dtype=store)

                def copy(x, start):
                    nb, low, lst = int(x[CX_BITS]), int(x[CX_LOW]), int(x[CX_LIST])
                    q = np.arange(1 << nb)
                    offs = [1 << b for b in range(low)] + [int(y) for y in c[lst: lst + nb - low]]
                    lds[:, int(x[CX_LDS]) + q] = arena[start[:, None] + _deposit(q, offs)]

                if c[CH_FCOPY]:
                    copy(c[CH_X:], src_t)
                for i, s in enumerate(st) if typ == 0 else ():
                    copy(s[CS_X:], base(s[CS_G:]) + at(2 + i))
                for i, s in enumerate(st):
                    k = np.arange(1 << (int(s[0]) & 255))
                    src, g, out = maps[i]
                    G = (lds[:, int(s[CS_X + CX_LDS]) + g[:, None] + k] if typ == 0 else
                         arena[(base(s[CS_G:]) + at(2 + i))[:, None, None] + g[:, None] + k])
                    S = (arena[src_t[:, None, None] + src[:, None] + k] if i == 0 and not c[CH_FCOPY] else
                         lds[:, int(s[CS_SRC]) + src[:, None] + k])
                    a = np.ldexp((S.astype(np.float64) * G).sum(2), shift[i])  # before it is rounded
                    largest[i] = max(largest[i], float(np.max(np.abs(a))))
                    v = a.astype(store)
                    assert np.isfinite(v).all()
                    if i + 1 < L:
                        lds[:, int(s[CS_DST]) + out] = v
                    else:
                        result[(out_t[:, None] + out) - off[int(c[CH_TC])]] = v
            flagged |= any(0.0 < m < TINY for m in largest[:-1])
            done.append((int(off[int(c[CH_TC])]), result, int(c[CH_TC]), e_total))
        for o, v, t, e in done:
            arena[o: o + len(v)] = v
            mx[t], ex[t] = np.max(np.abs(v.astype(np.float64))), e
    root = info["n_tensors"] - 1
    return float(arena[off[root]]), int(ex[root]), flagged


def off_by(m, e, om, oe):
    """Relative error of m * 2^e against om * 2^oe."""
    if om == 0.0 or m == 0.0:
        return 0.0 if om == m else math.inf
    return abs(math.ldexp(m / om, max(-2000, min(2000, e - oe))) - 1.0)


def listed_off_by(plan, w, om, oe):
    """The same of the plan's launch list (each weight leaf scaled to below 1,
    as the leaf kernel does)."""
    s = [math.frexp(float(max(abs(w[2 * v]), abs(w[2 * v + 1]))))[1] for v in range(len(w) // 2)]
    total, _ = pe.emulate(plan, np.ldexp(w, -np.repeat(s, 2)), np.float64 if plan.precision == "fp64" else np.float32)
    if total == 0 or om == 0.0:
        return 0.0 if total == om else math.inf
    return abs(float(total * Fraction(2) ** (sum(s) - oe) / Fraction(om)) - 1.0)


def fp32_lost():
    """Formulas whose chains, kept in a fixed range, lose every entry that the
    count needs although each stage's largest entry is ordinary."""
    for seed, s in ((52, 1e-7), (52, 1e-8), (52, 1e-9), (77, 1e-7)):
        pick = np.random.default_rng(seed).random((18, 1)) < 0.5
        yield wl.random_kcnf(18, 70, seed=seed).with_weights(np.where(pick, [0.5, 0.5 * s], [0.5 * s, 0.5]))
    f = wl.banded_3cnf(33, 99, 12, seed=53)
    for seed in (10, 15, 20, 33, 56):
        rng = np.random.default_rng(seed)
        yield f.with_weights(rng.uniform(0.5, 0.99, (f.n, 2)) * np.where(rng.random((f.n, 1)) < 0.5, [1, 1e-25], [1, 1]))


def test_chains_keep_what_the_launch_list_keeps():
    """Every tensor of these chains stays in range, and the count is right."""
    for q, f in enumerate(fp32_lost()):
        p = W.Plan(W.Network.from_formula(f), seed=0, precision="fp32")
        m, e, flagged = ranged(p, np.asarray(f.weights).reshape(-1))
        assert not flagged and off_by(m, e, *oracle.bucket(f)) <= tolerance(p), q


def skewed(seed):
    """A small formula with some literals of widely different weights."""
    rng = np.random.default_rng(seed)
    n = int(rng.integers(14, 36))
    f = (wl.random_kcnf(n, int(n * rng.uniform(2.5, 4.2)), seed=seed) if n < 20 and rng.random() < 0.5 else
         wl.banded_3cnf(n, int(n * rng.uniform(2.5, 4.0)), int(rng.integers(7, 13)), seed=seed))
    w = rng.uniform(0.1, 0.9, (n, 2))
    pick = rng.random(n) < rng.choice([0.3, 0.6, 1.0])
    w[pick, rng.integers(0, 2, int(pick.sum()))] *= 10.0 ** rng.uniform(*rng.choice([[-4, -1], [-12, -4], [-40, -20]]),
                                                                    int(pick.sum()))
    return f.with_weights(w)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_no_wrong_count_is_in_range(precision):
    """A replay that reports no intermediate out of range has the count,
    unless the launch list has lost it, too."""
    flags, wrong = 0, 0
    for seed in range(160):
        f = skewed(seed)
        p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision)
        if p.program()[1]["n_launches"] == 0:
            continue
        w = np.asarray(f.weights).reshape(-1)
        m, e, flagged = ranged(p, w)
        flags += flagged
        om, oe = oracle.bucket(f)
        if flagged or off_by(m, e, om, oe) <= tolerance(p):
            continue
        wrong += 1
        assert listed_off_by(p, w, om, oe) >= 0.5 * off_by(m, e, om, oe), (seed, m, e, om, oe)
    assert wrong <= 16, wrong  # the property is about counts that FP32 can hold
    assert flags <= 40, flags  # and a report is the exception


def out_of_range(precision, seed=0):
    """A formula whose chains lose the count and whose launch list keeps it."""
    f = wl.banded_3cnf(60, 210, 15, seed=3)
    small = 1e-60 if precision == "fp64" else 1e-9
    return f.with_weights(np.random.default_rng(seed).uniform(0.1, 0.9, (f.n, 2)) * [1.0, small])


def sliced_out_of_range(precision, group=2):
    """The same in some slices of a plan only: four slices, one of them zero."""
    f = wl.banded_3cnf(60, 180, 15, seed=5)
    small = 1e-60 if precision == "fp64" else 1e-9
    f = f.with_weights(np.random.default_rng(0).uniform(0.1, 0.9, (f.n, 2)) * [1.0, small])
    return f, W.Plan(W.Network.from_formula(f), seed=0, precision=precision, rank_cap=11, slice_group=group)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_out_of_range_cases_need_the_launch_list(precision):
    """What the device tests below count on: left to themselves the chains of
    these cases give a wrong count, they report it, and the launch list is
    right; of the sliced plan's slices some report and one does not."""
    for seed in range(2):
        f = out_of_range(precision, seed)
        p, w, (om, oe) = W.Plan(W.Network.from_formula(f), seed=0, precision=precision), f.weights.reshape(-1), oracle.bucket(f)
        m, e, flagged = ranged(p, w)
        assert flagged and off_by(m, e, om, oe) > 0.5 and listed_off_by(p, w, om, oe) <= tolerance(p)
    f, p = sliced_out_of_range(precision)
    assert p.n_slices == 4 and listed_off_by(p, f.weights.reshape(-1), *oracle.bucket(f)) <= tolerance(p)
    got = [ranged(p, f.weights.reshape(-1), eta) for eta in range(4)]
    assert [x[2] for x in got] == [True, False, True, True] and [x[0] == 0.0 for x in got] == [True, False, True, False]


def test_lift_keeps_products_finite():
    """A chain's tensors stay below 2^top, top bounded where a consumer
    multiplies them as they are stored."""
    seen = set()
    for precision in ("fp64", "fp32"):
        for f, kw in ((wl.banded_3cnf(80, 280, 18, seed=2), dict(block=4)), (wl.banded_3cnf(60, 210, 15, seed=1), {})):
            p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, **kw)
            prog, info = parse(p)
            nk = {int(t): int(d["nk"]) for d in prog["nodes"] for t in (d["ta"], d["tb"])}
            for typ, _, _, cf, cc, _, _, _ in prog["launches"]:
                for desc in prog["chains"][cf: cf + cc]:
                    c, n = prog["words"][int(desc):], CS_WORDS[int(typ)]
                    summed = sum(int(c[CH_WORDS + i * n]) & 255 for i in range(int(c[0])))
                    matrix = precision == "fp32" and nk.get(int(c[CH_TC]), 0) >= 4
                    top = 480 if precision == "fp64" else 56 if matrix else 126
                    assert int(c[CH_WORDS + CS_LIFT]) == top - summed
                    assert all(c[CH_WORDS + i * n + CS_LIFT] == 0 for i in range(1, int(c[0])))
                    seen.add(top)
    assert seen == {480, 126, 56}


@pytest.mark.gpu
def test_counts_in_range_on_device():
    """The formulas of the replay above."""
    for q, f in enumerate(fp32_lost()):
        p = W.Plan(W.Network.from_formula(f), seed=0, precision="fp32")
        assert same(W.wmc_contract(p), *oracle.bucket(f), tolerance(p)), q


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("small", [1.0, 1e-3, 1e-6])
def test_chains_that_feed_matrix_nodes(precision, small):
    """Chain outputs read by nodes with K >= 16, which multiply them as stored."""
    for f, kw in ((wl.banded_3cnf(80, 280, 18, seed=2), dict(block=4)),
                  (wl.banded_3cnf(150, 520, 18, seed=3), dict(block=4))):
        rng = np.random.default_rng(1)
        f = f.with_weights(rng.uniform(0.1, 0.9, (f.n, 2)) * np.where(rng.random((f.n, 1)) < 0.4, [1.0, small], [1, 1]))
        p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, **kw)
        assert p.program()[1]["n_chains"] > 0
        assert same(W.wmc_contract(p), *oracle.bucket(f), tolerance(p)), kw


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_out_of_range_solves(precision):
    """One solve, and a sliced plan's sums, per-slice values and resumed sums:
    the launch list's counts, whatever the slices that run side by side."""
    f = out_of_range(precision)
    p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision)
    v, (g, _) = W.wmc_contract(p), W.wmc_contract_profile(p)
    assert same(v, *oracle.bucket(f), tolerance(p)) and (v.mantissa, v.exp2) == (g.mantissa, g.exp2)
    assert W.wmc_contract_noalloc(p) == v
    first = None
    for group in (1, 2, 4):
        f, p = sliced_out_of_range(precision, group)
        v, (g, _) = W.wmc_contract(p), W.wmc_contract_profile(p)
        assert same(v, *oracle.bucket(f), tolerance(p)) and same(g, *oracle.bucket(f), tolerance(p))
        total, per = W.wmc_contract_slices(p, 0, 4, per_slice=True)
        assert total == v and per[2].mantissa == 0.0 and per[0].mantissa != 0.0
        state, half = W.wmc_slice_state(), []
        for _ in range(2):
            half.append(W.wmc_contract_resume(p, state, 2))
        assert half[1] == v and half[0] == W.wmc_contract_slices(p, 0, 2)
        first = first or (v, per)
        assert (v, per) == first, group


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_out_of_range_batches_and_servers(precision):
    """Beside ordinary instances, which keep their values bit for bit."""
    ordinary = [wl.banded_3cnf(60, 210, 15, seed=9), wl.random_kcnf(18, 60, seed=3)]
    sf, sp = sliced_out_of_range(precision)
    fs = [ordinary[0], out_of_range(precision, 0), sf, ordinary[1], out_of_range(precision, 1)]
    plans = [sp if f is sf else W.Plan(W.Network.from_formula(f), seed=0, precision=precision) for f in fs]
    refs = [oracle.bucket(f) for f in fs]
    calm = [W.Batch([plans[q]]).contract()[0] for q in (0, 3)]
    b = W.Batch(plans)
    ws = b.workspace()
    for flags in (0, W.BATCH_GRAPH, W.BATCH_GRAPH | W.BATCH_RESIDENT, W.BATCH_RESIDENT, W.BATCH_PERSISTENT,
                  W.BATCH_GRAPH | W.BATCH_RESIDENT):
        got = b.contract(ws=ws, flags=flags)
        for v, p, (om, oe) in zip(got, plans, refs):
            assert same(v, om, oe, tolerance(p)), flags
        assert [(got[q].mantissa, got[q].exp2) for q in (0, 3)] == [(v.mantissa, v.exp2) for v in calm], flags
    srv = W.Server(precision=precision, max_slots=8, hbm_budget_bytes=1 << 28, buffer_bytes=1 << 29)
    ids = [srv.register(p) for p in plans]
    for q in range(15):
        srv.submit(ids[q % 5], fs[q % 5].weights.reshape(-1), q)
    done = srv.drain()
    assert sorted(r.request_id for r in done) == list(range(15))
    for r in done:
        assert same(r.value, *refs[r.request_id % 5], tolerance(plans[r.request_id % 5])), r.request_id


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_out_of_range_batch_with_matrix_nodes(precision):
    """Instances with matrix nodes, some of which run again: each has what
    its plan's launch list gives alone, the others what they give alone."""
    f = wl.banded_3cnf(80, 280, 18, seed=2)
    small = 1e-60 if precision == "fp64" else 1e-9
    rng = np.random.default_rng(4)
    fs = [f, f.with_weights(rng.uniform(0.1, 0.9, (f.n, 2)) * [1.0, small]), out_of_range(precision),
          f.with_weights(rng.uniform(0.1, 0.9, (f.n, 2)))]
    plans = [W.Plan(W.Network.from_formula(g), seed=0, precision=precision, block=1 if q == 2 else 4)
             for q, g in enumerate(fs)]
    assert plans[0].image()[1]["n_gemms"] > 0 and plans[0].program()[1]["n_chains"] > 0
    lists = [W.wmc_contract_profile(p)[0] for p in plans]
    b = W.Batch(plans)
    ws = b.workspace()
    for flags in (0, W.BATCH_GRAPH | W.BATCH_RESIDENT, W.BATCH_GRAPH | W.BATCH_RESIDENT):
        for q, (v, p, g) in enumerate(zip(b.contract(ws=ws, flags=flags), plans, lists)):
            assert same(v, g.mantissa, g.exp2, tolerance(p)), (q, flags)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_many_slices_out_of_range(precision):
    """8192 slices, about half of them out of range, looked at 1024 and (in
    groups of 3) 1023 at a time: the values and sums do not depend on how the
    slices are grouped or on where a range begins."""
    first = None
    f, _ = sliced_out_of_range(precision)
    for group in (8, 3):
        p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, rank_cap=7, slice_group=group)
        assert p.n_slices == 8192 and p.program()[1]["n_launches"] > 0
        ws = W.workspace(p)
        total, per = W.wmc_contract_slices(p, 0, 8192, ws=ws, per_slice=True)
        assert same(total, *oracle.bucket(f), tolerance(p))
        assert total == W.wmc_contract(p, ws=ws) and total == W.wmc_contract(p, ws=ws)
        part, some = W.wmc_contract_slices(p, 1000, 2100, ws=ws, per_slice=True)
        assert some == per[1000:2100] and part == W.wmc_contract_slices(p, 1000, 2100, ws=ws)
        state = W.wmc_slice_state()
        for count in (1, 1500, 1000, 6000):
            v = W.wmc_contract_resume(p, state, count, ws=ws)
        assert v == total
        first = first or (total, per)
        assert (total, per) == first


def crowded():
    """A lattice whose chains report an intermediate out of range."""
    f = wl.grid_cnf(8, 14, 0.2, seed=2)
    return f.with_weights(np.random.default_rng(0).uniform(0.1, 0.9, (f.n, 2)) * [1.0, 1e-12])


def test_crowded_lattice_runs_again():
    f = crowded()
    p, w = W.Plan(W.Network.from_formula(f), seed=0, precision="fp32"), f.weights.reshape(-1)
    assert ranged(p, w)[2] and listed_off_by(p, w, *oracle.bucket(f)) <= tolerance(p)


@pytest.mark.gpu
@pytest.mark.parametrize("step_kib", [80, 96, 160, 320])
def test_requests_that_run_again_fit_the_staging(step_kib):
    """Many requests at once that run again, where the staging of a step
    bounds how many run side by side."""
    fs = [crowded(), wl.grid_cnf(8, 14, 0.2, seed=3)]
    plans = [W.Plan(W.Network.from_formula(f), seed=0, precision="fp32") for f in fs]
    refs = [oracle.bucket(f) for f in fs]
    srv = W.Server(precision="fp32", max_slots=64, hbm_budget_bytes=1 << 28, buffer_bytes=1 << 29,
                   step_bytes=step_kib << 10)
    ids = [srv.register(p) for p in plans]
    kind = [int(q % 8 == 7) for q in range(96)]
    for q, k in enumerate(kind):
        srv.submit(ids[k], fs[k].weights.reshape(-1), q)
    done = srv.drain()
    assert sorted(r.request_id for r in done) == list(range(96))
    for r in done:
        k = kind[r.request_id]
        assert same(r.value, *refs[k], tolerance(plans[k])), r.request_id


@pytest.mark.parametrize("rows,cols,ternary,seed,block,fused", [
    (14, 15, 0.122, 890, 6, False), (6, 16, 0.105, 606, 6, False), (6, 12, 0.155, 246, 5, False),
    (13, 15, 0.1, 7, 3, True), (9, 13, 0.1, 7, 2, True)])
def test_small_plan_keeps_its_launch_list_unless_chains_save_launches(rows, cols, ternary, seed, block, fused):
    """Row by row: matrix nodes leave chains only at the ends of the sweep."""
    f = wl.grid_cnf(rows, cols, ternary, seed=seed)
    p = W.Plan(W.Network.from_formula(f), kind="order", order=wl.row_major_order(rows, cols), block=block)
    assert (p.program()[1]["n_launches"] > 0) == fused
