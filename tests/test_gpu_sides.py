"""Every mesh side a plan accepts (2^a 3^b, a >= 2, 16..1024) has its own transform, field and post-pass
kernels: each side's multipoles against the oracle, with k edges that end below the Nyquist wavenumber
(the passes skip what lies beyond the last edge) and field groups that split +m / -m pairs.  Tolerances
are the parity tests' (per precision form)."""
from __future__ import annotations

import math

import numpy as np
import pytest

from tests.parity_util import assert_pole_parity, oracle_params, small_catalogs
from tests.test_gpu_sizes import _cube_catalog

pytestmark = pytest.mark.gpu

SMALL = [16, 24, 32, 36, 48, 64, 72, 96, 108, 128, 144]
LARGE = [192, 216, 256, 288, 324, 432, 512, 576, 648, 864, 972]


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n", SMALL)
def test_small_side_equals_oracle(gpu, n, prec):
    from oracle.estimator import multipoles
    from paper_1704_02357_amd import Plan
    L, obs = 320.0, (35.0, -20.0, -600.0)
    d, r = small_catalogs(2500, 12000, L, seed=3 * n)
    kn = math.pi * n / L
    # bins up to 0.55 and up to 1.7 Nyquist (past the corners' axis modes), 4 fields at a time and all at once
    for top, group in ((0.55, 4), (1.7, 0)):
        edges = np.linspace(0.0, top * kn, 5)
        plan = Plan(n, L, observer=obs, precision=prec, ell_max_hint=4, max_group=group)
        plan.paint(d, r)
        print(f"[case] side {n} prec={prec} top={top} group={group}", flush=True)
        got = plan.compute_multipoles(4, edges)
        plan.close()
        ref = multipoles(d, r, oracle_params(n, L, obs, 3, True, True), 4, edges)
        assert_pole_parity(got, ref, prec, f"side {n} top {top}")


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n", LARGE)
def test_large_side_equals_direct_sums(gpu, n, prec):
    """On-node cubes (exact on the mesh at any side), a low shell and one at 0.3 N, the last edge."""
    from oracle.direct import shell_modes, yamamoto_at_modes
    from oracle.estimator import default_params
    from paper_1704_02357_amd import Plan
    L = 4.0 * n
    obs = (0.13 * L, -0.21 * L, -1.7 * L)
    cat = _cube_catalog(n, L, 60, seed=n)
    lo = round((0.3 * n) ** 2)
    hi = lo + 1
    while len(shell_modes(n, np.array([lo, hi]), [0])[0]) < 1500:
        hi += 1
    thr, sel = np.array([1, 25, lo, hi], dtype=np.int64), [0, 2]
    edges = 2 * math.pi / L * np.sqrt(thr - 0.5)
    ells = [0, 2, 4]
    params = default_params(n, L, observer=obs, window=1, interlaced=False, compensated=True)
    modes, b = shell_modes(n, thr, sel)
    poles, counts, kmean = yamamoto_at_modes(cat, None, params, ells, modes, b, len(thr) - 1)
    print(f"[case] side {n} prec={prec} direct", flush=True)
    plan = Plan(n, L, observer=obs, window=1, interlaced=False, compensated=True, precision=prec, ell_max_hint=4,
                max_group=8)
    plan.paint(cat)
    got = plan.compute_multipoles(4, edges)
    plan.close()
    ref = {"poles": poles[:, sel], "n_modes": counts[sel].astype(np.int64), "k_mean": kmean[sel], "alpha": 0.0,
           "norm_I": got["norm_I"], "shot_noise": got["shot_noise"]}
    sub = {"poles": got["poles"][:, sel], "n_modes": got["n_modes"][sel], "k_mean": got["k_mean"][sel],
           "alpha": got["alpha"], "norm_I": got["norm_I"], "shot_noise": got["shot_noise"]}
    assert_pole_parity(sub, ref, prec, f"side {n}")
