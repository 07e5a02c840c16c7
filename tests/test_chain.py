"""The fused program (chains of contractions with their intermediates in
LDS): its descriptors replayed on the CPU, and the device against the
general launch list's oracle."""
import math

import numpy as np
import pytest

import oracle
import paper_2006_15512_amd as W
import wmc_workloads as wl
from plan_emulator import GEMM, LEAF, NODE, _pext, _sexp

CH_STAGES, CH_TILE_BITS, CH_F, CH_C, CH_TF, CH_TC, CH_FCOPY, CH_TILES, CH_X, CH_OUT, CH_SRC, CH_WORDS = (
    0, 1, 2, 4, 6, 7, 10, 11, 12, 16, 32, 48)
BITS = 16  # words per list of entry bit offsets
CS_SHAPE, CS_TBITS, CS_G, CS_TG, CS_SRC, CS_DST, CS_BIT, CS_X, CS_BIT_O, CS_PS, CS_PO, CS_QG, CS_QO = (
    0, 1, 2, 4, 5, 6, 8, 24, 40, 56, 58, 60, 62)
CS_WORDS = {0: 28, 3: 64}  # by launch type: short chains, chains of many tiles
CX_BITS, CX_LOW, CX_LDS, CX_LIST = 0, 1, 2, 3


def parse(plan):
    img, info = plan.program()
    out, at = {}, 0
    for key, dt, n in (("leaves", LEAF, info["n_leaves"]), ("nodes", NODE, info["n_nodes"]),
                       ("gemms", GEMM, info["n_gemms"]), ("words", np.dtype("<u4"), info["n_words"]),
                       ("recs", np.dtype(("<u4", (4,))), info["n_recs"]),
                       ("launches", np.dtype(("<i4", (8,))), info["n_launches"]),
                       ("chains", np.dtype("<u4"), info["n_chains"]),
                       ("off", np.dtype("<i8"), info["n_tensors"] if info["n_launches"] else 0)):
        out[key] = np.frombuffer(img, dt, count=n, offset=at)
        at += n * dt.itemsize
    return out, info


def _deposit(idx, offs):
    out = np.zeros(idx.shape, dtype=np.int64)
    for b, o in enumerate(offs):
        out |= ((idx >> b) & 1) * int(o)
    return out


def replay(plan, w):
    """(mantissa, exponent) of an unsliced plan's fused program, stage by stage
    as the kernel runs it, and the number of stages of its chains."""
    prog, info = parse(plan)
    store = np.float64 if plan.precision == "fp64" else np.float32
    arena = np.full(info["arena_elems"], np.nan, dtype=store)
    nt = info["n_tensors"]
    mx, ex = np.zeros(nt), np.zeros(nt, dtype=np.int64)
    off = prog["off"]
    for d in prog["leaves"]:
        e = np.arange(1 << int(d["rank"]))
        assert int(d["out"]) == off[int(d["tensor"])]
        if d["kind"] == 0:
            a = np.zeros(len(e), dtype=np.int64)
            for q in range(int(d["k"])):
                a |= ((e >> int(d["pos"][q])) & 1) << q
            v = np.where((a != int(d["falsify"])) | bool(d["taut"]), 1.0, 0.0)
        else:
            w0, w1 = w[2 * int(d["var"])], w[2 * int(d["var"]) + 1]
            v = np.where((e >> int(d["pos"][0])) & 1, w1, w0) if d["kind"] == 1 else np.array([w0 + w1])
            s = math.frexp(float(np.max(np.abs(v))))[1]
            v, ex[int(d["tensor"])] = np.ldexp(v, -s), s
        s = v.astype(store)
        arena[int(d["out"]): int(d["out"]) + len(e)] = s
        mx[int(d["tensor"])] = np.max(np.abs(s.astype(np.float64)))
    stages = []
    for typ, nf, nc, cf, cc, gi, rf, rc in prog["launches"]:
        done = []
        for d in prog["nodes"][nf: nf + nc] if typ != 2 else []:
            r = np.arange(1 << int(d["rc"]), dtype=np.uint64)
            nk = int(d["nk"])
            k = np.arange(1 << nk)
            A = arena[int(d["a"]) + (_pext(r, d["ra"], int(d["nra"])).astype(np.int64)[:, None] << nk | k)]
            B = arena[int(d["b"]) + (_pext(r, d["rb"], int(d["nrb"])).astype(np.int64)[:, None] << nk | k)]
            sh = _sexp(mx[int(d["ta"])]) + _sexp(mx[int(d["tb"])])
            v = np.ldexp((A.astype(np.float64) * B).sum(1), -sh).astype(store)
            done.append((int(d["c"]), v, int(d["tc"]), ex[int(d["ta"])] + ex[int(d["tb"])] + sh))
        assert typ != 2, "matrix nodes are not replayed here"
        # every tile of every chain of the launch is dealt exactly once
        want = {}
        for desc in prog["chains"][cf: cf + cc]:
            want[int(desc)] = np.zeros(1 << int(prog["words"][desc + CH_TILE_BITS]), dtype=int)
        for desc, blk, jb, _ in prog["recs"][rf: rf + rc]:
            want[int(desc)][int(blk) << int(jb): (int(blk) + 1) << int(jb)] += 1
        for n in want.values():
            assert np.all(n == 1)
        for desc in prog["chains"][cf: cf + cc]:
            c = prog["words"][desc:].astype(np.int64)
            L, ob = int(c[CH_STAGES]), int(c[CH_TILE_BITS])
            n = CS_WORDS[int(typ)]
            tiles = c[int(c[CH_TILES]):]
            st = [c[CH_WORDS + i * n: CH_WORDS + (i + 1) * n] for i in range(L)]
            base = lambda x: int(x[0]) + (int(x[1]) << 32)
            shift = [_sexp(mx[int(s[CS_TG])]) for s in st]
            shift[0] += _sexp(mx[int(c[CH_TF])])
            e_total = ex[int(c[CH_TF])] + sum(ex[int(s[CS_TG])] for s in st) + sum(shift)
            result = np.full(1 << len(plan.tensor(int(c[CH_TC]))[2]), np.nan, dtype=store)
            maps = []
            for i, s in enumerate(st):
                nk, np_, nq, tb = int(s[0]) & 255, (int(s[0]) >> 8) & 255, int(s[0]) >> 16, int(s[CS_TBITS])
                outs = s[CS_BIT_O:] if typ == 3 else c[CH_OUT:] if i + 1 == L else 1 << np.arange(16)
                if typ == 0:  # source in the low half, G in the high half
                    memory = i == 0 and not c[CH_FCOPY]
                    bits = [(int(c[CH_SRC + b]) if memory else int(s[CS_BIT + b]) & 0xFFFF, int(s[CS_BIT + b]) >> 16,
                             int(outs[b])) for b in range(tb)]
                else:
                    bits = [(int(s[CS_BIT + b]), int(s[CS_BIT + BITS + b]), int(outs[b])) for b in range(tb)]
                    bits += [(int(s[CS_PS + q]), 0, int(s[CS_PO + q])) for q in range(np_)]
                    bits += [(0, int(s[CS_QG + q]), int(s[CS_QO + q])) for q in range(nq)]
                e = np.arange(1 << len(bits))
                maps.append([_deposit(e, [x[j] for x in bits]) for j in range(3)])
                assert len(np.unique(maps[-1][2])) == len(e)
                stages.append((nk, np_, nq, i == 0, i + 1 == L, int(typ)))
            for t in np.array_split(np.arange(1 << ob), max(1, (1 << ob) // 32)):  # a few tiles at a time
                at = lambda q: _deposit(t, tiles[q * ob: (q + 1) * ob])
                src_t, out_t = base(c[CH_F:]) + at(0), base(c[CH_C:]) + at(1)
                lds = np.full((len(t), 65536 // np.dtype(store).itemsize), np.nan, dtype=store)

                def copy(x, start):
                    """The part of an operand each tile reads, into its LDS region."""
                    nb, low, at = int(x[CX_BITS]), int(x[CX_LOW]), int(x[CX_LIST])
                    q = np.arange(1 << nb)
                    offs = [1 << b for b in range(low)] + [int(y) for y in c[at: at + nb - low]]
                    lds[:, int(x[CX_LDS]) + q] = arena[start[:, None] + _deposit(q, offs)]

                if c[CH_FCOPY]:
                    copy(c[CH_X:], src_t)
                for i, s in enumerate(st) if typ == 0 else ():
                    copy(s[CS_X:], base(s[CS_G:]) + at(2 + i))
                for i, s in enumerate(st):
                    k = np.arange(1 << (int(s[CS_SHAPE]) & 255))
                    src, g, out = maps[i]
                    G = (lds[:, int(s[CS_X + CX_LDS]) + g[:, None] + k] if typ == 0 else
                         arena[(base(s[CS_G:]) + at(2 + i))[:, None, None] + g[:, None] + k])
                    S = (arena[src_t[:, None, None] + src[:, None] + k] if i == 0 and not c[CH_FCOPY] else
                         lds[:, int(s[CS_SRC]) + src[:, None] + k])
                    v = np.ldexp((S.astype(np.float64) * G).sum(2), -shift[i]).astype(store)
                    assert not np.isnan(v).any()
                    if i + 1 < L:
                        lds[:, int(s[CS_DST]) + out] = v
                    else:
                        to = (out_t[:, None] + out) - off[int(c[CH_TC])]
                        assert np.isnan(result[to]).all()
                        result[to] = v
            assert not np.isnan(result).any()
            done.append((int(off[int(c[CH_TC])]), result, int(c[CH_TC]), e_total))
        for o, v, t, e in done:  # a launch's outputs never land on its inputs
            arena[o: o + len(v)] = v
            mx[t], ex[t] = np.max(np.abs(v.astype(np.float64))), e
    root = info["n_tensors"] - 1
    return float(arena[off[root]]), int(ex[root]), stages


CASES = [dict(f=lambda: wl.random_kcnf(18, 60, seed=3), kw={}),
         dict(f=lambda: wl.banded_3cnf(60, 210, 15, seed=1), kw={}),
         dict(f=lambda: wl.banded_3cnf(80, 280, 18, seed=2), kw=dict(block=2)),
         dict(f=lambda: wl.banded_3cnf(110, 380, 25, seed=2), kw=dict(block=3)),
         dict(f=lambda: wl.grid_cnf(7, 14, 0.2, seed=4), kw=dict(block=3)),
         dict(f=lambda: wl.grid_cnf(9, 13, 0.1, seed=7), kw=dict(kind="order", order=wl.row_major_order(9, 13))),
         dict(f=lambda: wl.grid_cnf(9, 13, 0.1, seed=7), kw=dict(kind="order", order=wl.row_major_order(9, 13), block=2))]


def tolerance(plan):
    """FP32: one rounding of 2^-24 per stored intermediate of the tree."""
    return 1e-12 if plan.precision == "fp64" else 2.0 ** -24 * plan.stats()["n_nodes"]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_program_replay_equals_oracle(precision):
    """The chains' words, replayed tile by tile with every entry written
    once and read only after it was written, give the oracle's count; the
    cases reach every summed size in both kinds of chain."""
    seen = set()
    for case in CASES:
        f = case["f"]()
        p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, **case["kw"])
        m, e, stages = replay(p, np.asarray(f.weights).reshape(-1))
        seen |= set(stages)
        om, oe = oracle.bucket(f)
        if om == 0.0:
            assert m == 0.0
        else:
            assert abs(math.ldexp(m / om, e - oe) - 1.0) <= tolerance(p)
    assert {nk for nk, _, _, _, _, typ in seen if typ == 0} == {0, 1, 2, 3}
    assert {nk for nk, _, _, _, _, typ in seen if typ == 3} == {0, 1, 2, 3}
    assert {(a, b) for _, a, b, _, _, typ in seen if typ == 3} >= {(0, 0), (1, 0), (1, 1)}


def same(v, m, e, tol):
    return v.mantissa == 0.0 if m == 0.0 else abs(math.ldexp(v.mantissa / m, v.exp2 - e) - 1.0) <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_chains_on_device_equal_oracle(precision):
    """wmc_contract on the fused program: the cases of the replay, and the
    general launch list (the profile runs it) beside it."""
    for case in CASES:
        f = case["f"]()
        p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, **case["kw"])
        assert p.program()[1]["n_launches"] > 0
        om, oe = oracle.bucket(f)
        v, (g, _) = W.wmc_contract(p), W.wmc_contract_profile(p)
        assert same(v, om, oe, tolerance(p)) and same(g, om, oe, tolerance(p)), case["kw"]
        if precision == "fp64" and not case["kw"]:  # the same sums in the same order
            assert (v.mantissa, v.exp2) == (g.mantissa, g.exp2)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("small", [1e-4, 1e-15, 1e-60])
def test_chain_out_of_range_runs_the_launch_list(precision, small):
    """Weights so uneven that forced assignments make intermediates of a
    chain tiny (an intermediate below the tiles' range sends the whole call
    to the launch list, which scales every tensor): wherever the launch list
    itself gives the oracle's count, the call does.  (Entries below 2^-126, in
    FP64 2^-1022, of their tensor's largest are zero on either path, which
    the smallest of these weights reach.)"""
    for seed in range(3):
        f = wl.banded_3cnf(60, 210, 15, seed=seed)
        rng = np.random.default_rng(seed)
        w = np.where(rng.random((f.n, 1)) < 0.5, small, 1.0) * rng.uniform(0.1, 0.9, (f.n, 2)) * [1.0, small]
        g = f.with_weights(w)
        om, oe = oracle.bucket(g)
        p = W.Plan(W.Network.from_formula(g), seed=0, precision=precision)
        v, (general, _) = W.wmc_contract(p), W.wmc_contract_profile(p)
        fits = same(general, om, oe, tolerance(p))
        assert fits or small < (1e-4 if precision == "fp32" else 1e-15), seed
        assert same(v, om, oe, tolerance(p)) or not fits, (seed, v, om, oe)


@pytest.mark.gpu
@pytest.mark.parametrize("precision,small", [("fp64", 1e-15), ("fp32", 1e-4)])
def test_out_of_range_chains_in_batches_and_servers(precision, small):
    """The same weights in a batch (eager and replayed, beside an ordinary
    instance) and served (several in flight): where the launch list gives the
    oracle's count, both do, and the ordinary instance keeps its value."""
    fs, refs = [wl.banded_3cnf(60, 210, 15, seed=9)], []
    for seed in range(3):
        f = wl.banded_3cnf(60, 210, 15, seed=seed)
        rng = np.random.default_rng(seed)
        fs.append(f.with_weights(np.where(rng.random((f.n, 1)) < 0.5, small, 1.0) * rng.uniform(0.1, 0.9, (f.n, 2)) *
                                 [1.0, small]))
    plans = [W.Plan(W.Network.from_formula(f), seed=0, precision=precision) for f in fs]
    refs = [oracle.bucket(f) for f in fs]
    b = W.Batch(plans)
    ws = b.workspace()
    for flags in (0, W.BATCH_GRAPH, W.BATCH_GRAPH | W.BATCH_RESIDENT):
        for v, p, (om, oe) in zip(b.contract(ws=ws, flags=flags), plans, refs):
            assert same(v, om, oe, tolerance(p)), flags
    srv = W.Server(precision=precision, max_slots=8, hbm_budget_bytes=1 << 28, buffer_bytes=1 << 29)
    ids = [srv.register(p) for p in plans]
    for q in range(12):
        srv.submit(ids[q % 4], np.asarray(fs[q % 4].weights).reshape(-1), q)
    done = srv.drain()
    assert sorted(r.request_id for r in done) == list(range(12))
    for r in done:
        om, oe = refs[r.request_id % 4]
        assert same(r.value, om, oe, tolerance(plans[r.request_id % 4])), r.request_id


@pytest.mark.parametrize("name,fused", [("grid24", False), ("grid24_minfill", True)])
def test_plan_that_chains_hardly_help_keeps_its_launch_list(name, fused):
    """A plan whose bytes go to nodes with K >= 16 has no fused program; the
    same formula on a tree of K <= 8 nodes has one."""
    import bench
    f, pkw, _, _ = bench.workload(name)
    pkw = dict(pkw)
    plan, _ = bench.make_plan(W, f, "fp64", pkw.pop("block"), pkw)
    assert (plan.program()[1]["n_launches"] > 0) == fused
