"""Pairs whose separation on a periodic axis lies on both sides of half the box, within the cutoff (boxes
of four nodes, cutoff 2.02), in every class of bead counts, against the oracle's substeps."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests.common import gpu_sim, oracle_sim
from workloads import configs as WC
from workloads.configs import FREESLIP, PERIODIC, Box, MDParams, Replica

pytestmark = pytest.mark.gpu


def _beads(box, n, rng):
    """n beads anywhere, 0.8 apart through the periodic faces, every tenth half a box from
    another but for a few hundredths."""
    size, r = np.array([box.nx, box.ny, box.nz], float), []
    while len(r) < n:
        p = rng.uniform(0.0, size)
        if r and len(r) % 10 == 0:
            p = r[rng.integers(len(r))] + [0.0, 2.0 + rng.uniform(-0.03, 0.03), 0.1]
        p[0] = np.clip(p[0], 1.5, box.nx - 2.5)
        d = np.array(r).reshape(-1, 3) - p
        d[:, 1:] -= 4.0 * np.round(d[:, 1:] / 4.0)
        if not len(d) or np.min(np.sum(d * d, axis=1)) > 0.64:
            r.append(p)
    return np.array(r)


@pytest.mark.parametrize("x", [FREESLIP, PERIODIC], ids=["x_faces", "periodic"])
@pytest.mark.parametrize("n,nx", [(20, 12), (60, 16), (100, 24), (200, 40), (400, 70), (700, 110), (1100, 170)])
def test_half_a_box_apart(n, nx, x):
    box = Box(nx, 4, 4, (x, PERIODIC, PERIODIC))
    md = MDParams(M=3, eps=1e-6, eps_w=1e-6, k_bond=0.0, f_drive=0.0)
    r = _beads(box, n, np.random.default_rng(n))
    rep = Replica(box, [1] * n, 23)
    from paper_0710_1272_amd import lbmd as B
    ora = oracle_sim(rep, md, beads=r, step0=2)
    u_o, _ = O.interp(box, ora.f, ora.r)
    r_o, v_o = ora.r.copy(), ora.v.copy()
    _, flags_o = O.md_substeps(box, md, rep.chain_len, r_o, v_o, u_o, 2, rep.seed)
    with gpu_sim([rep], md, WC.STORE_F64, beads=r, step0=2) as sim:
        sim.couple(B.LB_COUPLE_INTERP)
        sim.md_step()
        r_g, v_g = sim.beads(allow_unstable=True)
        word, _ = sim.status()
    # the same FP64 formulas in another order of rounding; the steepest pair (0.8 apart) turns a
    # position's last bit (2e-14 at 110) into 1e2 times that in its force, three times over
    assert word == flags_o
    assert np.max(np.abs(v_g - v_o)) < 1e-8 * max(1.0, float(np.max(np.abs(v_o))))
    assert np.max(np.abs(r_g - r_o)) < 1e-8
    assert np.max(np.abs(v_o)) > 1e-3
