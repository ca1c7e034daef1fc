"""The constraint solve of a rigid chain (one tridiagonal system, log2 levels of cyclic reduction)
at the chain lengths where a level more or less is taken and where the rows fill a wave, against
the oracle's substeps."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from tests.common import gpu_sim, oracle_sim
from workloads import configs as WC
from workloads import generate as G
from workloads.configs import FREESLIP, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


# a substep's constraint forces carry the solve's rounding, a few 1e-15 of the bond length, and the
# convergence tolerance |s^2 - b^2| <= 1e-12 b^2 met by both sides from different roundings; five
# substeps of a stiff contact model stay below 1e-11, as for the other lengths tested
@pytest.mark.parametrize("chains", [[2], [3], [4], [5], [9], [17], [33], [2, 2, 2], [64, 2], [65], [128, 1], [129], [200]],
                         ids=lambda c: "_".join(map(str, c)))
def test_rigid_rows(chains):
    box = Box(60, 60, 60, (FREESLIP,) * 3, (), 1.0)
    md = WC.paper_polymer(rigid=1, kappa_phi=0.05, eps=1.0, eps_w=1.0)
    beads = np.zeros((0, 3))
    grow = dataclasses.replace(MDParams(), sigma=1.75)
    for k, n in enumerate(chains):
        new = G.grow_chain(box, grow, n, np.random.default_rng(11 + k), existing=beads if len(beads) else None,
                           cis_only=False)
        beads = np.concatenate([beads, new])
    rep = Replica(box, chains, 43)
    rho, u = G.random_small_flow(box, 6, du=0.01)
    from paper_0710_1272_amd import lbmd as B
    ora = oracle_sim(rep, md, rho, u, beads=beads, step0=9)
    u_o, _ = O.interp(box, ora.f, ora.r)
    r_o, v_o = ora.r.copy(), ora.v.copy()
    fbar_o, flags_o = O.md_substeps(box, md, chains, r_o, v_o, u_o, 9, rep.seed)
    with gpu_sim([rep], md, WC.STORE_F64, rho, u, beads=beads, step0=9) as sim:
        sim.couple(B.LB_COUPLE_INTERP)
        sim.md_step()
        r, v = sim.beads()
        _, fbar, _ = sim.coupling()
        word, _ = sim.status()
    scale = max(1.0, float(np.max(np.abs(v_o))))
    assert word == flags_o == 0
    assert np.max(np.abs(r - r_o)) < 1e-11
    assert np.max(np.abs(v - v_o)) < 1e-11 * scale
    assert np.max(np.abs(fbar - fbar_o)) < 1e-11 * scale
