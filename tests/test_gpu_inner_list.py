"""One lane a bead: the substeps' inner list against the oracle where it can go wrong: as many entries
as there are slots and more, more than it holds, beads that move past its margin within a step (it is
taken again) and past the Verlet list's (both are), the smallest and largest bead counts."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests.common import gpu_sim, oracle_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import FREESLIP, PERIODIC, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


# Single precision rounds a coordinate's force to 6e-8 of at most about 10 (eps = 0.05) in each of 20
# substeps of h = 1/20, in double precision 1e-16: v is off by 20 h 10 6e-8 = 6e-7 and 1e-15, and a
# difference grows up to 50-fold over the step (two oracle runs 1e-7 apart).
@pytest.mark.parametrize("storage,tol", [(WC.STORE_F64, 1e-11), (WC.STORE_F32, 1e-4)], ids=["f64", "f32"])
@pytest.mark.parametrize("periodic", [False, True], ids=["faces", "periodic"])
@pytest.mark.parametrize("speed", [0.0, 0.3, 0.7], ids=lambda v: f"v{v}")
@pytest.mark.parametrize("n,lanes,spacing", [(27, 1, 1.02), (257, 0, 1.02), (300, 0, 0.95), (512, 0, 0.95), (512, 0, 1.4)])
def test_inner_list_substeps(n, lanes, spacing, speed, periodic, storage, tol):
    box = Box(24, 20, 20, ((PERIODIC if periodic else FREESLIP),) * 3, (), 1.0)
    # rc = 1.01: at a spacing of 0.95 a bead in the middle has 18 others within the inner radius, at
    # 1.02 six
    md = MDParams(M=20, eps=0.05, sigma=0.9, eps_w=0.05, sigma_w=0.5, k_bond=0.0, f_drive=0.0)
    rng = np.random.default_rng(n)
    i = np.arange(n)
    r = 3.0 + spacing * np.stack([i % 8, (i // 8) % 8, i // 64], axis=1) + rng.uniform(-0.01, 0.01, (n, 3))
    if periodic:
        r[:, 0] += 18.0  # across the boundary
    v = speed * rng.choice([-1.0, 1.0], (n, 1)) * np.array([[1.0, 0.2, 0.1]])
    rep = Replica(box, [1] * n, 53)
    rho, u = G.random_small_flow(box, 6, du=0.01)
    from paper_0710_1272_amd import lbmd as B
    ora = oracle_sim(rep, md, rho, u, beads=r, v=v, step0=4)
    u_o, _ = O.interp(box, ora.f, ora.r)
    r_o, v_o = ora.r.copy(), ora.v.copy()
    fbar_o, flags_o = O.md_substeps(box, md, rep.chain_len, r_o, v_o, u_o, 4, rep.seed)
    with gpu_sim([rep], md, storage, rho, u, beads=r, v=v, step0=4, md_lanes=lanes) as sim:
        assert sim.md_lanes == 1
        sim.couple(B.LB_COUPLE_INTERP)
        sim.md_step()
        r_g, v_g = sim.beads()
        _, fb_g, _ = sim.coupling()
        word, _ = sim.status()
    scale = max(1.0, float(np.max(np.abs(v_o))))
    assert word == flags_o == 0
    assert np.max(np.abs(r_g - r_o)) < tol
    assert np.max(np.abs(v_g - v_o)) < tol * scale
    assert np.max(np.abs(fb_g - fbar_o)) < tol * scale
