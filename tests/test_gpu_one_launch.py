"""A coupled step of one small box in one launch against its halves in launches of their own
(interpolation, substeps, lattice step, spread), around the edges of what takes it: boxes that do not
fill a block or a 64-node chunk, the smallest and largest bead counts of each lane count, several beads
on one node, the last box size inside and the first outside, single steps and graphs."""
from __future__ import annotations

import numpy as np
import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads.configs import FREESLIP, Box, MDParams, Replica

pytestmark = pytest.mark.gpu

F64, F32, F16, BF16 = WC.STORE_F64, WC.STORE_F32, WC.STORE_F16, WC.STORE_BF16
# Both ways form the same sums in the same order, so that only a compiler's choice of a fused
# product can differ: the last bit of an operation, of which a population's update has about 50, and
# 16-bit storage may then round the other way, one unit of the element.
POP = {F64: 64 * 2.0**-52, F32: 64 * 2.0**-23, F16: 2.0**-10, BF16: 2.0**-7}


def _beads(box, n, rng):
    """n beads on a straight zigzag through the box, in both lower and the upper corner, the last
    three on one node."""
    i = np.arange(n)
    r = np.stack([1.0 + (i * 1.2) % (box.nx - 3), 1.0 + (1.2 * (i * 1.2 // (box.nx - 3))) % (box.ny - 3),
                  1.0 + 1.3 * ((i * 1.2 // (box.nx - 3)) // ((box.ny - 3) / 1.2))], axis=1)
    r += rng.uniform(-0.05, 0.05, r.shape)
    wall = box.walls[0]
    r[:, 0] += np.where((r[:, 0] > wall[0] - 1.5) & (r[:, 0] < wall[1] + 1.5), 5.0, 0.0)
    if n > 3:
        r[0] = [0.2, 0.3, 0.1]
        r[1] = [box.nx - 1.2, box.ny - 1.3, box.nz - 1.1]
        r[-3:] = r[-1] + rng.uniform(-0.02, 0.02, (3, 3))
    return r


@pytest.mark.parametrize("storage", [F64, F32, F16, BF16], ids=["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("size,n,steps", [((37, 13, 11), 1, 1), ((37, 13, 11), 9, 3), ((64, 16, 8), 32, 17), ((50, 21, 9), 33, 3),
                                          ((65, 20, 19), 65, 17), ((48, 40, 20), 128, 1), ((48, 40, 20), 129, 3),
                                          ((48, 40, 20), 256, 2), ((48, 40, 20), 257, 2), ((128, 128, 80), 12, 1),
                                          ((129, 128, 80), 12, 1)], ids=lambda p: str(p).replace(" ", ""))
def test_one_launch_step_equals_halves(size, n, steps, storage):
    if size[0] >= 128 and storage in (F64, BF16):
        pytest.skip("the size limit is tested in FP32 and FP16")
    box = Box(*size, (FREESLIP,) * 3, ((size[0] // 2, size[0] // 2 + 1, 3, 5, 3, 5),), 1.0)
    rng = np.random.default_rng(n)
    # soft, short-ranged beads: the chain may be placed anywhere, and overlapping beads stay put
    md = MDParams(M=5, eps=0.0, eps_w=0.0, k_bond=0.0, f_drive=0.0)
    rep = Replica(box, [1] * n, 47)
    beads = _beads(box, n, rng)
    x = np.arange(box.nodes) / box.nodes
    rho = 1.0 + 0.02 * np.sin(40 * x)
    u = 0.02 * np.stack([np.cos(30 * x), np.sin(50 * x), np.cos(70 * x)])
    from paper_0710_1272_amd import lbmd as B
    with gpu_sim([rep], md, storage, rho, u, beads=beads) as one:
        one.step(steps)
        f1, (r1, v1), c1, s1 = one.populations(), one.beads(), one.coupling(), one.status()
    with gpu_sim([rep], md, storage, rho, u, beads=beads) as two:
        for _ in range(steps):
            two.couple(B.LB_COUPLE_INTERP)
            two.md_step()
            two.step(1, coupled=False)
            two.couple(B.LB_COUPLE_SPREAD)
        f2, (r2, v2), c2, s2 = two.populations(), two.beads(), two.coupling(), two.status()
    assert s1 == s2
    bead_tol = (1e-13 if storage == F64 else 1e-6) * steps
    assert np.max(np.abs(r1 - r2)) <= bead_tol * max(size)
    assert np.max(np.abs(v1 - v2)) <= bead_tol
    assert np.array_equal(c1[2], c2[2])
    dev = np.max(np.abs(f2)) if storage in (F64, F32) else 0.05
    assert np.max(np.abs(f1 - f2)) <= steps * POP[storage] * dev
