"""A prepared plan stays within the bytes that plan_footprint announces, the list of post-pass tiles included."""
from __future__ import annotations

import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(64, 0), (216, 1), (432, 1)])
def test_prepared_plan_within_footprint(gpu, n, prec):
    """432^3 in FP64 has single-line tiles: 91 000 of them, when the last edge lies past the corner modes."""
    from paper_1704_02357_amd import Plan
    from paper_1704_02357_amd.pkm import plan_footprint
    L, nb, particles = 1000.0, 20, 10000
    plan = Plan(n, L, precision=prec, ell_max_hint=4)
    plan.prepare(4, np.linspace(0.0, 1.8 * math.pi * n / L, nb + 1), particles)
    used = plan.stats()["device_bytes"]
    plan.close()
    room = plan_footprint(n, L, 4, nb + 1, particles, precision=prec, ell_max_hint=4)
    print(f"[footprint] side {n} prec={prec} used {used} of {room}", flush=True)
    assert used <= room
