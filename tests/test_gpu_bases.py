"""Odd multipoles and the Cartesian decomposition at sides with kernels of their own (12-point, 6-point and
short lines), with field groups that cut the +m / -m and monomial pairs: small sides against the oracle, large
ones against the even spherical call on the same painted plan.  Tolerances are those of the tests of either
call at powers of two."""
from __future__ import annotations

import functools
import math

import numpy as np
import pytest

from tests.parity_util import assert_pole_parity, oracle_params, small_catalogs
from tests.test_gpu_cartesian import assert_per_ell

pytestmark = pytest.mark.gpu

L, OBS = 300.0, (40.0, -25.0, -650.0)


def _edges(n):
    return np.linspace(0.0, 1.2 * math.pi * n / L, 6)


@functools.lru_cache(maxsize=1)
def _oracle(n):
    from oracle.estimator import all_multipoles, multipoles
    d, r = small_catalogs(2500, 12000, L, seed=5 * n)
    params = oracle_params(n, L, OBS, 3, True, True)
    return d, r, all_multipoles(d, r, params, 5, _edges(n)), multipoles(d, r, params, 4, _edges(n))


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,max_group", [(24, 0), (36, 7), (72, 7), (96, 0), (108, 7), (128, 7)])
def test_small_side_equals_oracle(gpu, n, max_group, prec):
    from paper_1704_02357_amd import Plan
    d, r, ref_all, ref_even = _oracle(n)
    print(f"[case] bases side {n} group={max_group} prec={prec}", flush=True)
    plan = Plan(n, L, observer=OBS, precision=prec, ell_max_hint=4, max_group=max_group)
    plan.paint(d, r)
    odd = plan.compute_multipoles_all(5, _edges(n))
    cart = plan.compute_multipoles(4, _edges(n), basis=1)
    plan.close()
    assert_pole_parity(odd, ref_all, prec, f"all l, side {n}")
    assert_per_ell(cart, ref_even, prec, f"Cartesian, side {n}")


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n", [216, 288, 324, 432, 648])
def test_large_side_equals_even_spherical(gpu, n, prec):
    from paper_1704_02357_amd import Plan
    d, r = small_catalogs(20000, 100000, L, seed=5 * n)
    print(f"[case] bases side {n} prec={prec}", flush=True)
    plan = Plan(n, L, observer=OBS, precision=prec, ell_max_hint=4, max_group=7)
    plan.paint(d, r)
    even = plan.compute_multipoles(4, _edges(n))
    cart = plan.compute_multipoles(4, _edges(n), basis=1)
    odd = plan.compute_multipoles_all(5, _edges(n))
    plan.close()
    assert_per_ell(cart, even, prec, f"Cartesian, side {n}")
    assert_per_ell(dict(odd, poles=odd["poles"][0::2]), even, prec, f"all l, side {n}")
    assert np.isfinite(odd["poles"]).all()
