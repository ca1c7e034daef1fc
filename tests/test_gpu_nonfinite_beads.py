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
