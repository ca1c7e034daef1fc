"""Solvent-free steps enqueued together (the step counter handed from launch to launch) against single
ones, around the graph length and with replicas without beads."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import FREESLIP, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [True, False], ids=["graph", "direct"])
@pytest.mark.parametrize("steps", [2, 3, 16, 17, 18])
@pytest.mark.parametrize("beads", [[12], [0, 7, 0, 30]], ids=["one", "some_empty"])
def test_no_solvent_run_equals_single_steps(beads, steps, graph):
    from paper_0710_1272_amd import lbmd as B
    md = MDParams()
    box = Box(24, 16, 16, (FREESLIP,) * 3, (), 1.0)
    reps = [Replica(box, [n] if n else [], 61 + k) for k, n in enumerate(beads)]
    r = np.concatenate([G.grow_chain(box, md, n, np.random.default_rng(n), cis_only=False) for n in beads if n])
    flags = 0 if graph else B.LB_CFG_NO_GRAPH
    with gpu_sim(reps, md, WC.STORE_F32, beads=r, step0=3, flags=flags) as a, \
            gpu_sim(reps, md, WC.STORE_F32, beads=r, step0=3, flags=flags) as b:
        for _ in range(2):
            a.step(steps, hydro=False)
            for _ in range(steps):
                b.step(1, hydro=False)
            a.step(1)
            b.step(1)
        assert a.status() == b.status() == (0, 3 + 2 * (steps + 1))
        for k, n in enumerate(beads):
            if not n:
                continue
            for x, y in zip(a.beads(k), b.beads(k)):
                assert np.array_equal(x, y)
            ta, tb = a.transloc(k), b.transloc(k)
            assert ta.keys() == tb.keys() and all(np.array_equal(ta[key], tb[key]) for key in ta)
