"""What a fused program may take in memory."""
import numpy as np
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
