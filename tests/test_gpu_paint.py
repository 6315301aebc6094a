"""Painted meshes against tap sums in FP64: sides whose blocks paint one, two and four tiles of a row,
every window, catalogs in mesh order and with repeated positions (whole runs of one tile in the count), a
dense clump beside lone particles, positions on cell faces and outside the box."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _catalog(n, L, seed):
    from synth import Catalog
    rng = np.random.default_rng(seed)
    h = L / n
    lone = rng.random((9001, 3)) * L
    clump = (np.array([0.31, 0.52, 0.77]) + 0.02 * rng.random((3011, 3))) * L
    faces = np.repeat(rng.integers(0, 2 * n, (150, 3)) * (0.5 * h), 13, axis=0)
    outside = rng.uniform(-1.2, 2.3, (257, 3)) * L
    edges = np.repeat(np.array([[0.0, 0.0, 0.0], [L - 1e-9 * L, 0.0, 0.5 * h], [0.5 * h, L - 0.5 * h, L - h]]), 70, axis=0)
    ordered = lone[np.lexsort((lone[:, 2] // h, lone[:, 1] // h, lone[:, 0] // h))]
    pos = np.concatenate((ordered, clump, faces, outside, edges)) - 0.5 * L
    m = len(pos)
    return Catalog(pos, rng.uniform(0.3, 2.0, m), np.full(m, 1e-3))


def _taps(cat, sign, n, L, window, shift):
    from oracle.mesh import axis_taps, mesh_coords
    u = mesh_coords(cat.pos, L, (-0.5 * L,) * 3, n) + (0.5 if shift else 0.0)
    idx, val = [], []
    for ix, wx in axis_taps(u[:, 0], window):
        for iy, wy in axis_taps(u[:, 1], window):
            for iz, wz in axis_taps(u[:, 2], window):
                idx.append(((ix % n) * n + iy % n) * n + iz % n)
                val.append(sign * cat.w * wx * wy * wz)
    return np.concatenate(idx), np.concatenate(val)


def _deterministic_quantum(cats, n, L):
    """Largest value of 1/sc for 8-node tiles: 8 (largest tile count) (largest weight) / sc <= 2^60, sc a power
    of two and not half of what that allows."""
    from oracle.mesh import mesh_coords
    t = np.concatenate([np.floor(mesh_coords(c.pos, L, (-0.5 * L,) * 3, n)).astype(np.int64) % n // 8 for c in cats])
    most = np.unique((t[:, 0] * n + t[:, 1]) * n + t[:, 2], return_counts=True)[1].max()
    return 2.0 * 8.0 * most * max(np.max(c.w) for c in cats) * 2.0 ** -60


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n,window,det", [(36, 3, False), (72, 1, False), (72, 2, True), (72, 3, False), (256, 1, True),
                                          (256, 2, False), (256, 3, False), (432, 3, False), (512, 1, False),
                                          (512, 2, False), (512, 3, False), (512, 3, True)])
def test_painted_meshes(gpu, n, window, det, prec):
    from oracle.catalog import catalog_scalars
    from paper_1704_02357_amd import Plan
    L = 700.0
    d, r = _catalog(n, L, n + window), _catalog(n, L, 7 * n + window)
    alpha = catalog_scalars(d, r, L)["alpha"]
    print(f"[case] paint side {n} window {window} prec={prec} deterministic={det}", flush=True)
    plan = Plan(n, L, window=window, interlaced=True, precision=prec, deterministic=det)
    plan.paint(d, r)
    for which, shift in ((0, False), (1, True)):
        got = plan.read_buffer(which).reshape(-1)
        idx, val = (np.concatenate(x) for x in zip(_taps(d, 1.0, n, L, window, shift),
                                                   _taps(r, -alpha, n, L, window, shift)))
        nodes, inv = np.unique(idx, return_inverse=True)
        exp, mag, taps = np.bincount(inv, val), np.bincount(inv, np.abs(val)), np.bincount(inv)
        # FP64: up to some 6000 roundings of 2^-53 of a node's magnitude; FP32: exact fixed-point sums of a
        # tile, rounded and added for at most 8 blocks, and the store's rounding; deterministic: half a quantum
        # a tap
        tol = 1e-12 if prec else 10 * 2.0 ** -24
        quantum = _deterministic_quantum((d, r), n, L) if det else 0.0
        err = np.max(np.abs(got[nodes] - exp) - tol * mag - 0.5 * quantum * taps)
        print(f"[paint] mesh {which} nodes {len(nodes)} excess {err:.2e}", flush=True)
        assert err <= 1e-13
        assert np.count_nonzero(got) <= len(nodes)
    plan.close()
