"""Requests of many k bins, whose post-pass histograms leave no room in the LDS of a compute unit for a
block's usual lines: up to the limit a plan's shape sets they run, above it they are refused.  Small sides
against the oracle; large ones against a coarse request whose bins are unions of the fine ones, with the
parity tests' tolerances."""
from __future__ import annotations

import math

import numpy as np
import pytest

from tests.parity_util import TOL, assert_pole_parity, oracle_params, small_catalogs

pytestmark = pytest.mark.gpu

L, OBS = 500.0, (40.0, -60.0, -900.0)


def _edges(n, nb):
    return np.linspace(0.0, 1.73 * math.pi * n / L, nb + 1)


@pytest.mark.parametrize("n,prec,ell,nb,shape", [
    (64, 1, 4, 3300, dict(tile_post=1)),  # 6 of 8 lines a block
    (64, 0, 4, 3300, dict(tile_post=1)),
    (72, 1, 16, 1400, dict(tile_post=1)),  # eleven rows of bins in one group
    (96, 0, 4, 3200, dict(tile_post=1)),
])
def test_many_bins_equal_oracle(gpu, n, prec, ell, nb, shape):
    from oracle.estimator import multipoles
    from paper_1704_02357_amd import Plan
    d, r = small_catalogs(2500, 12000, L, seed=n + nb)
    edges = _edges(n, nb)
    plan = Plan(n, L, observer=OBS, precision=prec, ell_max_hint=ell, shape=shape)
    plan.paint(d, r)
    print(f"[case] bins {nb} side {n} prec={prec} l<={ell}", flush=True)
    got = plan.compute_multipoles(ell, edges)
    plan.close()
    assert_pole_parity(got, multipoles(d, r, oracle_params(n, L, OBS, 3, True, True), ell, edges), prec,
                       f"{nb} bins, side {n}")


@pytest.mark.parametrize("n,prec,ell,nb", [
    (144, 1, 4, 3150), (192, 1, 4, 1300), (192, 1, 4, 2250), (288, 1, 4, 2900), (192, 0, 4, 2830), (768, 0, 4, 3000),
    (1024, 0, 4, 2500),
    (432, 1, 8, 2460),  # seven rows: the thresholds stay in global memory
])
def test_many_bins_equal_coarse_bins(gpu, n, prec, ell, nb):
    from paper_1704_02357_amd import Plan
    d, r = small_catalogs(20000, 100000, L, seed=n + nb)
    plan = Plan(n, L, observer=OBS, precision=prec, ell_max_hint=ell)
    plan.paint(d, r)
    fine_edges, step = _edges(n, nb), nb // 10
    print(f"[case] bins {nb} side {n} prec={prec} l<={ell}", flush=True)
    fine = plan.compute_multipoles(ell, fine_edges)
    coarse = plan.compute_multipoles(ell, fine_edges[::step])
    plan.close()
    counts = fine["n_modes"][: nb // step * step].reshape(-1, step)
    assert np.array_equal(counts.sum(1), coarse["n_modes"])
    raw = coarse["poles"][0] + coarse["shot_noise"]
    for row, (f, c) in enumerate(zip(fine["poles"], coarse["poles"])):
        f = np.where(counts > 0, f[: counts.size].reshape(counts.shape), 0.0)
        err = np.abs((f * counts).sum(1) / counts.sum(1) - c) / np.maximum(np.abs(c), raw)
        print(f"[bins] row {row} err {err.max():.2e}", flush=True)
        assert err.max() <= TOL[prec]


@pytest.mark.parametrize("n,prec,most", [(192, 1, 2258), (144, 1, 3160), (512, 0, 2601)])
def test_bin_limit_of_the_default_shape(gpu, n, prec, most):
    from paper_1704_02357_amd import Plan, PkmError
    plan = Plan(n, L, observer=OBS, precision=prec, ell_max_hint=4, max_group=4)
    plan.prepare(4, _edges(n, most), 100)
    with pytest.raises(PkmError, match="too many k bins"):
        plan.prepare(4, _edges(n, most + 1), 100)
    plan.close()
