"""One context taken through every kind of step in turn, coupled steps in one launch, bit for bit as
with coupled steps in launches of their own: the marks and step words of either buffer parity are
right after the counter moved another way.  And the one-launch step with the angular term, rigid chains
and the caller's lanes a bead against its halves."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import MDParams, Replica

pytestmark = pytest.mark.gpu

BOX = WC.pore_box(48, 24, 24)


def _case(md, n=40):
    rep = Replica(BOX, [n], 5)
    rho, u = G.random_small_flow(BOX, 3, du=0.01)
    v = np.array([-0.1, 0.03, 0.02]) + np.zeros((n, 3))  # a bead changes its node every few steps
    return rep, dict(rho=rho, u=u, beads=G.replica_beads(rep, md), v=v)


def _state(sim):
    return (sim.populations(), *sim.beads(), *sim.coupling(), np.array(sim.status()))


@pytest.mark.parametrize("graph", [True, False], ids=["graph", "launches"])
@pytest.mark.parametrize("step0", [0, -1, 2**40], ids=["0", "-1", "2^40"])
@pytest.mark.parametrize("storage", [WC.STORE_F32, WC.STORE_F16], ids=["f32", "f16"])
def test_steps_of_every_kind_in_turn(storage, step0, graph):
    from paper_0710_1272_amd import lbmd as B
    md = MDParams()
    rep, init = _case(md)
    flags = 0 if graph else B.LB_CFG_NO_GRAPH
    out = []
    for kw in ({}, dict(block_size=256)):
        with gpu_sim([rep], md, storage, step0=step0, flags=flags, **init, **kw) as sim:
            assert sim.one_launch == (not kw)
            seen = []
            for kind, n in (("c", 3), ("l", 1), ("c", 1), ("n", 3), ("c", 2), ("l", 2), ("n", 1), ("c", 17), ("n", 2),
                            ("l", 3), ("c", 1), ("h", 1), ("c", 2), ("c", 1)):
                if kind == "h":
                    sim.couple(B.LB_COUPLE_INTERP)
                    sim.md_step()
                    sim.step(n, coupled=False)
                    sim.couple(B.LB_COUPLE_SPREAD)
                else:
                    sim.step(n, coupled=kind == "c", hydro=kind != "n")
                seen.append(_state(sim))
            out.append(seen)
    for k, (a, b) in enumerate(zip(*out)):
        for x, y in zip(a, b):
            assert np.array_equal(x, y), k


@pytest.mark.parametrize("storage", [WC.STORE_F64, WC.STORE_F32], ids=["f64", "f32"])
@pytest.mark.parametrize("model", ["harmonic", "rigid", "angle", "rigid_angle"])
@pytest.mark.parametrize("n,lanes", [(20, 16), (20, 2), (60, 4), (200, 2)])
def test_models_and_lanes_as_halves(model, n, lanes, storage):
    from paper_0710_1272_amd import lbmd as B
    md = WC.paper_polymer() if "rigid" in model else MDParams()
    md.kappa_phi = 0.5 if "angle" in model else 0.0
    rep, init = _case(md, n)
    out = []
    for halves in (False, True):
        with gpu_sim([rep], md, storage, md_lanes=lanes, **init) as sim:
            assert sim.one_launch and sim.md_lanes == lanes
            if not halves:
                sim.step(3)
            for _ in range(3 if halves else 0):
                sim.couple(B.LB_COUPLE_INTERP)
                sim.md_step()
                sim.step(1, coupled=False)
                sim.couple(B.LB_COUPLE_SPREAD)
            out.append(_state(sim))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
