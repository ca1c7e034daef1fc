"""Streamed or ordinary population stores on both sides of every limit: size, and number of replicas."""
from __future__ import annotations

import pytest

from tests.common import gpu_sim
from workloads import configs as WC
from workloads.configs import Box, MDParams, Replica

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,side,storage,streamed", [
    (1, 128, WC.STORE_F32, False), (1, 129, WC.STORE_F32, False), (1, 132, WC.STORE_F32, True),
    (7, 64, WC.STORE_F32, False), (8, 64, WC.STORE_F32, True), (7, 66, WC.STORE_F32, False), (7, 70, WC.STORE_F32, True),
    (28, 48, WC.STORE_F16, False), (32, 48, WC.STORE_F16, True),
], ids=lambda p: str(p))
def test_store_policy(n, side, storage, streamed):
    rep = Replica(Box(side, side, side), [], 1)
    with gpu_sim([rep] * n, MDParams(), storage) as sim:
        assert sim.launch_shape()["nt_stores"] == streamed
