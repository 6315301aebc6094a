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
    (1024, 0, 4, 107),  # so that two blocks share a CU: likewise
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


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,top", [(16, 1.2), (16, 3.3), (64, 2.5), (1024, 1.2)])
def test_few_modes_equal_direct_sums(gpu, n, top, prec):
    """Last edges of a few fundamental modes: fewer post-pass tiles than XCDs."""
    from oracle.direct import shell_modes, yamamoto_at_modes
    from oracle.estimator import default_params
    from paper_1704_02357_amd import Plan
    from tests.test_gpu_sizes import _cube_catalog
    box = 4.0 * n
    obs = (0.13 * box, -0.21 * box, -1.7 * box)
    cat = _cube_catalog(n, box, 12, seed=n)
    thr = np.array([1, math.ceil(top * top)], dtype=np.int64)
    edges = 2 * math.pi / box * np.sqrt(thr - 0.5)
    params = default_params(n, box, observer=obs, window=1, interlaced=False, compensated=True)
    modes, b = shell_modes(n, thr, [0])
    poles, counts, kmean = yamamoto_at_modes(cat, None, params, [0, 2], modes, b, 1)
    print(f"[case] few modes side {n} top {top} prec={prec}", flush=True)
    plan = Plan(n, box, observer=obs, window=1, interlaced=False, compensated=True, precision=prec, ell_max_hint=2)
    plan.paint(cat)
    got = plan.compute_multipoles(2, edges)
    plan.close()
    ref = {"poles": poles, "n_modes": counts.astype(np.int64), "k_mean": kmean, "alpha": 0.0,
           "norm_I": got["norm_I"], "shot_noise": got["shot_noise"]}
    assert_pole_parity(dict(got, alpha=0.0), ref, prec, f"side {n} top {top}")


def test_many_bins_replayed_as_graph(gpu):
    """Blocks of fewer lines inside a captured batch: every replay, with eager work between, equals the
    synchronous calls."""
    import torch
    from paper_1704_02357_amd import Batch, Plan
    from synth import Catalog
    n, nb = 64, 3300
    d, r = (Catalog(*(torch.as_tensor(a, device="cuda") for a in (c.pos, c.w, c.nbar)))
            for c in small_catalogs(2500, 12000, L, seed=7))
    torch.cuda.synchronize()
    edges = _edges(n, nb)
    plan = Plan(n, L, observer=OBS, precision=1, ell_max_hint=4, shape=dict(tile_post=1),
                stream=torch.cuda.Stream())
    plan.paint(d, r)
    ref = plan.compute_multipoles(4, edges)
    plan.prepare(4, edges, 14500)
    batch = Batch()
    batch.add(plan, d, r)
    print("[case] many bins in a graph", flush=True)
    for _ in range(3):
        batch.run(use_graph=True)
        got = batch.result(0)
        assert_pole_parity(got, ref, 1, "replay")
        torch.randn(1 << 20, device="cuda").sum().item()
    batch.close()
    plan.close()
