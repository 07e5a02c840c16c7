"""What a fused program may take in memory."""
import pytest

import paper_2006_15512_amd as W
import wmc_workloads as wl


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_refused_program_takes_no_memory(precision):
    """A program whose own placement does not fit the plan's cap is not kept,
    and a batch of the plan reserves the plan's arena."""
    net = W.Network.from_formula(wl.banded_3cnf(42, 146, 14, seed=2))
    cap = W.Plan(net, seed=0, block=3, precision=precision).stats()["arena_bytes"]
    p = W.Plan(net, seed=0, block=3, precision=precision, mem_cap_bytes=cap)
    st = p.stats()
    assert p.program()[1]["n_launches"] == 0 and st["arena_bytes"] <= cap
    _, info = W.Batch([p]).image()
    assert info["arena_elems"] * info["elem"] == st["arena_bytes"]


def test_programs_add_little_to_a_large_workspace():
    """Eight arenas side by side, each of which a fused program would take
    beyond the launch list's: together they stay within 64 MiB more, beside
    the descriptors."""
    f = wl.banded_3cnf(185, 621, 31, seed=80)
    p = W.Plan(W.Network.from_formula(f), seed=1, block=3, rank_cap=21, slice_group=16)
    st = p.stats()
    assert st["slice_group"] == 8
    descriptors = len(p.image()[0]) + len(p.program()[0])
    assert st["workspace_bytes"] - 8 * st["arena_bytes"] <= (64 << 20) + 2 * descriptors + (1 << 20)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch_counts_the_launches_it_makes(precision):
    """The fused programs' launches where they run, the launch lists' where
    the programs' image would take more than a quarter of the workspace (a
    plan of 1024 small slices)."""
    f = wl.banded_3cnf(60, 180, 15, seed=5)
    p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision)
    n = p.program()[1]["n_launches"]
    assert 0 < n < p.stats()["n_launches"] - 3
    assert n + 3 <= W.Batch([p]).n_launches <= 2 * n + 3
    p = W.Plan(W.Network.from_formula(f), seed=0, precision=precision, rank_cap=8)
    b = W.Batch([p])
    assert p.n_slices == 1024 and p.program()[1]["n_launches"] > 0
    assert b.n_launches >= p.stats()["n_launches"]


@pytest.mark.parametrize("formulas,kw,fused", [
    (lambda: [wl.random_kcnf(12, 40, seed=i) for i in range(100)], {}, False),
    (lambda: [wl.grid_cnf(12, 14, 0.1, seed=i) for i in range(12)], dict(block=3), False),
    (lambda: [wl.banded_3cnf(110, 380, 25, seed=i) for i in (2, 3)], dict(block=3, rank_cap=17), False),
    (lambda: [wl.batch_instance(i) for i in range(24)], {}, True),
    (lambda: [wl.grid_cnf(16, 18, 0.1, seed=1)], dict(block=2), True)])
def test_batch_runs_chains_only_where_they_pay(formulas, kw, fused):
    """Batches that fill the device node by node keep their launch lists."""
    plans = [W.Plan(W.Network.from_formula(f), seed=0, **kw) for f in formulas()]
    assert any(p.program()[1]["n_launches"] for p in plans)
    b = W.Batch(plans)
    assert (b.n_launches < b.image()[1]["n_launches"] + 2) == fused


@pytest.mark.gpu
def test_resident_programs_leave_room_for_a_large_request():
    """A structure whose region takes all that the launch lists' images leave
    is served, though the fused programs of structures registered before it
    were kept in that room; those structures go on being served."""
    f, g = wl.grid_cnf(10, 20, 0.2, seed=2), wl.grid_cnf(16, 20, 0.1, seed=2)
    small = [W.Plan(W.Network.from_formula(f), seed=q, precision="fp32") for q in range(5)]
    large = W.Plan(W.Network.from_formula(g), seed=0, precision="fp32")
    budget = large.stats()["arena_bytes"] + int(1.3 * sum(len(p.image()[0]) for p in small + [large]))
    srv = W.Server(precision="fp32", max_slots=8, hbm_budget_bytes=budget, buffer_bytes=budget + (64 << 20))
    ids = [srv.register(p) for p in small]
    srv.submit(ids[0], f.weights.reshape(-1), 1)
    first = srv.wait(5.0)
    srv.submit(srv.register(large), g.weights.reshape(-1), 2)
    done = srv.wait(5.0)
    assert [r.request_id for r in done] == [2]
    assert abs(done[0].value.log2_abs - W.wmc_contract(large).log2_abs) < 1e-4
    for q, s in enumerate(ids):
        srv.submit(s, f.weights.reshape(-1), 10 + q)
    done = sorted(srv.drain(), key=lambda r: r.request_id)
    assert [r.request_id for r in done] == list(range(10, 15))
    assert all(abs(r.value.log2_abs - first[0].value.log2_abs) < 1e-4 for r in done)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_served_alone_and_in_a_burst(precision):
    """A structure whose requests run the fused program while they are few and
    the launch list while they are many: the same values, wmc_contract's."""
    f = wl.grid_cnf(10, 16, 0.1, seed=2)
    p = W.Plan(W.Network.from_formula(f), kind="order", order=wl.row_major_order(10, 16), block=3, precision=precision)
    v = W.wmc_contract(p)
    srv = W.Server(precision=precision, max_slots=64, hbm_budget_bytes=1 << 31, buffer_bytes=3 << 30)
    s = srv.register(p)
    for n in (1, 3, 200, 2):
        for q in range(n):
            srv.submit(s, f.weights.reshape(-1), q)
        done = srv.drain()
        assert sorted(r.request_id for r in done) == list(range(n))
        assert all((r.value.mantissa, r.value.exp2) == (v.mantissa, v.exp2) for r in done), n
