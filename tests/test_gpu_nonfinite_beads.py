"""A bead whose position is not finite sets LB_ERR_NONFINITE and leaves the other beads alone, also
beads with more neighbours than a list holds (they go through every bead of the box)."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads.configs import FREESLIP, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


def _substeps(box, md, storage, r, **kw):
    from paper_0710_1272_amd import lbmd as B
    with gpu_sim([Replica(box, [1] * len(r), 3)], md, storage, beads=r, **kw) as sim:
        sim.couple(B.LB_COUPLE_INTERP)
        sim.md_step()
        rr, vv = sim.beads(allow_unstable=True)
        return rr, vv, sim.status()[0]


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("n", [90, 180, 300], ids=["four_lanes", "two_lanes", "one_lane"])
@pytest.mark.parametrize("storage", [WC.STORE_F64, WC.STORE_F32], ids=["f64", "f32"])
def test_longer_lists_than_fit(storage, n, value):
    box = Box(24, 24, 24, (FREESLIP,) * 3)
    # beads on top of each other, without repulsion: all of them neighbours of all
    md = MDParams(M=3, eps=0.0, k_bond=0.0, f_drive=0.0)
    rng = np.random.default_rng(n)
    r = 12.0 + rng.uniform(-0.7, 0.7, (n, 3))
    r[n // 2] = [3.0, 3.0, 3.0]
    bad = r.copy()
    bad[n // 2] = value
    r0, v0, w0 = _substeps(box, md, storage, r)
    r1, v1, w1 = _substeps(box, md, storage, bad)
    rest = np.arange(n) != n // 2
    assert w0 == 0 and w1 & 4
    assert np.isfinite(r1[rest]).all()
    assert np.array_equal(r0[rest], r1[rest]) and np.array_equal(v0[rest], v1[rest])


WALL = Box(20, 12, 12, (FREESLIP,) * 3, ((9, 10, 4, 7, 0, 11),))
OPEN = Box(20, 12, 12, (FREESLIP,) * 3, ((9, 10, 0, 11, 0, 11),))


@pytest.mark.parametrize("rigid", [0, 1], ids=["beads", "rigid_model"])
@pytest.mark.parametrize("storage", [WC.STORE_F64, WC.STORE_F32], ids=["f64", "f32"])
@pytest.mark.parametrize("box,at,axis,value", [
    (WALL, (3.0, 1.0, 6.0), 0, np.nan),   # nowhere along x: at no wall
    (WALL, (8.2, 1.0, 6.0), 1, np.nan),   # no y: in front of the wall all the same
    (WALL, (8.2, 1.0, 6.0), 2, np.nan),
    (WALL, (8.2, 1.0, 6.0), 1, np.inf),
    (OPEN, (9.5, 6.0, 6.0), 2, np.nan),   # in a pore as high as the box for any z
    (OPEN, (9.5, 6.0, 6.0), 1, np.inf),
], ids=["x", "y", "z", "y_inf", "pore_z", "pore_y_inf"])
def test_walls(box, at, axis, value, storage, rigid):
    """Beads at a wall in one wave with the one that is nowhere; its other coordinates feel the wall
    and the drive as those of a bead in its place do, and only a bead inside the wall is reported so."""
    md = WC.paper_polymer(rigid=rigid, kappa_phi=0.0, M=1, k_bond=0.0, eps=0.0, eps_w=1e-3, sigma_w=0.5, f_drive=0.02)
    r = np.array([[8.2, 6.0, 6.0], at, [9.5, 5.5, 3.0], [11.0, 2.0, 9.0]])
    bad = r.copy()
    bad[1, axis] = value
    r0, v0, w0 = _substeps(box, md, storage, r)
    r1, v1, w1 = _substeps(box, md, storage, bad)
    rest = [0, 2, 3]
    assert w0 == 0 and w1 & 4
    assert np.array_equal(r0[rest], r1[rest]) and np.array_equal(v0[rest], v1[rest])
    if axis == 0:
        assert not w1 & 1
    else:
        assert v1[1, 0] == v0[1, 0]
        assert bool(w1 & 1) == (box is OPEN)  # x inside the slab, and no place in the pore's section
