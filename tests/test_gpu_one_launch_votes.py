"""One-launch coupled steps whose bead step runs in a few waves of its workgroup, with fast beads, so
that the kept Verlet list is voted stale at the start of most steps: bitwise the same twice, and as
the halves in launches of their own."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import MDParams, Replica

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12, 33, 100])
def test_few_bead_waves(n):
    box = WC.pore_box(48, 24, 24)
    md = MDParams()
    rng = np.random.default_rng(n)
    r = G.replica_beads(Replica(box, [n], 7), md)
    # the whole chain drifts by about skin / 2 in two steps, away from the wall
    v = np.array([-0.2, 0.0, 0.0]) + 0.05 * rng.standard_normal(r.shape)
    rep = Replica(box, [n], 7)
    from paper_0710_1272_amd import lbmd as B
    runs = []
    for halves in (False, False, True):
        with gpu_sim([rep], md, WC.STORE_F64, beads=r, v=v) as sim:
            if not halves:
                sim.step(8)
            for _ in range(8 if halves else 0):
                sim.couple(B.LB_COUPLE_INTERP)
                sim.md_step()
                sim.step(1, coupled=False)
                sim.couple(B.LB_COUPLE_SPREAD)
            runs.append((sim.populations(), *sim.beads(), sim.status()))
    a, b, h = runs
    assert a[3] == (0, 8) and b[3] == a[3] and h[3] == a[3]
    for k in range(3):
        assert np.array_equal(a[k], b[k])
    # FP64 roundings (1e-16 an operation, some 100 operations a substep, 160 substeps) and their growth
    # in collisions stay far below this; a pair missed or a stale list does not
    assert np.max(np.abs(a[1] - r)) > 0.5
    assert np.max(np.abs(a[0] - h[0])) < 1e-10 and np.max(np.abs(a[1] - h[1])) < 1e-9
