"""(k, mu) power at sides around the length of a thread's walk along y, with a slanted line of sight, mu edges
that modes hit exactly, and as many cells as a call takes: mode counts exactly, powers against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from tests.parity_util import TOL, oracle_params, small_catalogs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,los,nk,nmu", [(16, (0.0, 0.0, 1.0), 3, 1), (24, (1.0, 0.0, 0.0), 6, 5),
                                          (36, (0.6, 0.0, -0.8), 9, 10), (72, (0.0, -0.6, 0.8), 307, 10),
                                          (96, (0.0, 1.0, 0.0), 40, 20)])
def test_kmu_cells(gpu, n, los, nk, nmu, prec):
    from oracle.global_los import pkmu
    from paper_1704_02357_amd import Plan
    L = 300.0
    d, r = small_catalogs(3000, 20000, L, seed=n)
    kedges = np.linspace(0.0, 1.8 * np.pi * n / L, nk + 1)
    muedges = np.linspace(0.0, 1.0, nmu + 1)
    print(f"[case] kmu side {n} prec={prec} cells {nk} x {nmu}", flush=True)
    plan = Plan(n, L, precision=prec, los=los)
    plan.paint(d, r)
    pk, nm = plan.kmu_global(kedges, muedges)
    plan.close()
    pref, nref = pkmu(d, r, oracle_params(n, L, (0.0, 0.0, 0.0), 3, True, True), kedges, muedges, los)
    assert np.array_equal(nm, nref)
    ok = nref > 0
    raw = np.abs(pref) + 1.0 / (3000 / L ** 3)
    assert np.max(np.abs(pk[ok] - pref[ok]) / raw[ok]) < TOL[prec]
