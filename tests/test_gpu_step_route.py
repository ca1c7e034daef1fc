"""Which coupled steps run in one launch: both sides of every limit, and the launch shape a caller
names is that of coupled steps too, with the same bits."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import FREESLIP, PERIODIC, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


def _case(n=40, size=(48, 24, 24), bc=(FREESLIP,) * 3, kT=0.0, **md):
    box = Box(*size, bc, ((size[0] // 2, size[0] // 2 + 1, 4, 6, 4, 6),), 1.0, 1.0, kT)
    rng = np.random.default_rng(n)
    r = rng.uniform([1.0, 1.0, 1.0], [size[0] // 2 - 2.0, size[1] - 2.0, size[2] - 2.0], (n, 3))
    return Replica(box, [1] * n, 11), MDParams(M=4, eps=0.0, eps_w=0.0, k_bond=0.0, f_drive=0.0, **md), r


@pytest.mark.parametrize("one,case,kw", [
    (True, {}, {}),
    (True, dict(n=1), {}), (True, dict(n=256), {}), (False, dict(n=257), {}),
    (True, dict(n=200), dict(md_lanes=2)), (False, dict(n=12), dict(md_lanes=1)), (False, dict(n=300), dict(md_lanes=2)),
    (False, dict(bc=(FREESLIP, PERIODIC, FREESLIP)), {}), (False, dict(kT=1e-4), {}), (False, dict(stencil=1), {}),
    (False, {}, dict(obs_every=2, obs_capacity=4)),
    (False, {}, dict(block_size=128)), (False, {}, dict(mapping=1)), (False, {}, dict(xcd_order=-1)),
], ids=lambda p: str(p).replace(" ", ""))
def test_route(one, case, kw):
    rep, md, r = _case(**case)
    with gpu_sim([rep], md, WC.STORE_F32, beads=r, **kw) as sim:
        assert sim.one_launch == one


def test_two_replicas_and_none():
    rep, md, r = _case()
    with gpu_sim([rep, rep], md, WC.STORE_F32, beads=np.concatenate([r, r])) as sim:
        assert not sim.one_launch
    with gpu_sim([Replica(rep.box, [], 1)], md, WC.STORE_F32) as sim:
        assert not sim.one_launch


@pytest.mark.parametrize("storage", [WC.STORE_F64, WC.STORE_F32, WC.STORE_F16, WC.STORE_BF16],
                         ids=["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("rigid", [0, 1], ids=["harmonic", "rigid"])
def test_named_shape_is_used_and_changes_no_bit(storage, rigid):
    box = WC.pore_box(64, 32, 32)
    md = WC.paper_polymer() if rigid else MDParams()
    r = G.replica_beads(Replica(box, [60], 5), md)
    rep = Replica(box, [60], 5)
    rho, u = G.random_small_flow(box, 3, du=0.01)
    out = []
    for kw in ({}, dict(block_size=128, mapping=2), dict(block_size=256, mapping=4), dict(block_size=512, xcd_order=16)):
        with gpu_sim([rep], md, storage, rho, u, beads=r, **kw) as sim:
            assert sim.one_launch == (not kw)
            if kw:
                shape = sim.launch_shape()
                assert shape["block"] == kw["block_size"]
                assert shape["mapping"] == {0: "flat", 2: "rows", 4: "flat2"}[kw.get("mapping", 0)]
            sim.step(18)
            out.append((sim.populations(), *sim.beads(), *sim.coupling(), np.array(sim.status())))
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("storage", [WC.STORE_F64, WC.STORE_F32, WC.STORE_F16], ids=["f64", "f32", "f16"])
@pytest.mark.parametrize("n", [12, 100])
def test_autotune_times_the_step_that_runs(n, storage):
    """The tuned context takes the one launch where that is far the faster (12 beads: by a fifth or
    more), and goes on from the state it was given: bit for bit as an untuned context with its lanes."""
    from paper_0710_1272_amd import lbmd as B
    box = WC.pore_box(64, 32, 32)
    md = MDParams(M=5, k_bond=2.0, eps=2e-3, eps_w=2e-3)
    rep = Replica(box, [n], 5)
    r = G.replica_beads(rep, md)
    rho, u = G.random_small_flow(box, 3, du=0.01)
    with gpu_sim([rep], md, storage, rho, u, beads=r, flags=B.LB_CFG_AUTOTUNE) as a:
        lanes, one = a.md_lanes, a.one_launch
        assert a.status() == (0, 0)
        first = (a.populations(), *a.beads())
        a.step(19)
        end = (a.populations(), *a.beads(), np.array(a.status()))
    with gpu_sim([rep], md, storage, rho, u, beads=r, md_lanes=lanes) as b:
        assert all(np.array_equal(x, y) for x, y in zip(first, (b.populations(), *b.beads())))
        b.step(19)
        assert all(np.array_equal(x, y) for x, y in zip(end, (b.populations(), *b.beads(), np.array(b.status()))))
    if n == 12:
        assert one and lanes > 1
