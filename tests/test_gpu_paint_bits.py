"""FP32 meshes sum the taps of a painting block in 64-bit fixed point, scaled by the particles that may meet on
a node: blocks of one, two and four tiles of a row keep the same small remainders."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 256, 512])
def test_remainders_of_cancelling_weights(gpu, n):
    """Four neighbouring tiles of 256 particles each, half of weight 1 and half of -(1 - 2^-52) on one node a
    tile.  With every tap a multiple of 2^-52 the 128 pairs leave 2^-45 exactly; a scale for the block's 512 or
    1024 particles with no more bits than one for a tile's 256 would round them away."""
    from paper_1704_02357_amd import Plan
    from synth import Catalog
    L, pairs = float(n), 128
    nodes = np.array([[9, 10, 32 + 8 * t + 3] for t in range(4)])
    pos = np.repeat(nodes + 0.25, pairs, axis=0) - 0.5 * L  # (u = node + 1/4)
    nbar = np.full(len(pos), 1e-3)
    data = Catalog(pos, np.ones(len(pos)), nbar)
    rand = Catalog(pos, np.full(len(pos), 1.0 - 2.0 ** -52), nbar)
    print(f"[case] paint bits side {n}", flush=True)
    plan = Plan(n, L, window=1, interlaced=False, compensated=False, precision=0, shape=dict(paint_tile=8))
    plan.paint(data, rand)
    mesh = plan.read_buffer(0).reshape(n, n, n)
    plan.close()
    assert np.array_equal(mesh[tuple(nodes.T)], np.full(4, pairs * 2.0 ** -52, dtype=np.float32))
    assert np.count_nonzero(mesh) == 4
