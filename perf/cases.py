"""Performance cases of the multipole estimator: the estimates that programs using this
framework run, through its public entry points, from the smallest survey meshes to 1024^3.

Three kinds of pass:

  estimate   paint a catalog and measure P_l(k): `Plan.paint` + `Plan.compute_multipoles`
             (call "sync"), or `Plan.enqueue` + `Plan.finish` on a prepared plan (call "async").
             Catalogs are a survey (galaxies and randoms in a cone around the line of sight), a
             periodic box, or one weighted object on every mesh node (Gaussian mocks).
  kmu        paint a periodic box and bin |F_0|^2 in (k, mu) about a fixed line of sight.
  batch      several survey mocks of uneven size as one `Batch` unit replayed as a HIP graph.
  fft        the library's 3D transform, forward and back, on a caller's real mesh.

Inputs are drawn on the GPU from the seed.  The FP32 form's multipoles carry the rounding of
FP32 meshes and transforms; they are returned as float32 values, the FP64 form's as float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1704_02357_amd import Batch, Plan
from paper_1704_02357_amd.pkm import nonuniform_mu_edges, wedges

# Mesh sides the cases are drawn from: 2^a 3^b, power-of-two and radix-3 sizes alike.
SIZES = (48, 64, 72, 96, 108, 128, 144, 192, 216, 256, 288, 324, 384, 432, 512, 576, 648, 768)
LISTED_COST = 47 * 1024 ** 3       # transforms x cells of the largest listed estimate
STATE_BYTES = 6.0e10               # device bytes a drawn case's plan may hold


def _estimate(name, nmesh, box, n_data, n_rand, *, window=3, interlaced=True, compensated=True, ell_max=4,
              precision=0, call="async", catalog="survey", host=False, max_group=0, dk=0.01, mu_bins=0):
    return dict(name=name, kind="estimate", catalog=catalog, nmesh=nmesh, box=float(box), n_data=n_data,
                n_rand=n_rand, window=window, interlaced=interlaced, compensated=compensated, ell_max=ell_max,
                precision=precision, call=call, host=host, max_group=max_group, dk=dk, mu_bins=mu_bins)


def listed():
    return [
        # the plain FP64 method on a small survey: the smallest call, bound by launches
        _estimate("survey_64_cic_f64", 64, 1000, 30000, 300000, window=2, interlaced=False, precision=1, call="sync"),
        # a covariance mock read from files: host (numpy) catalogs handed to the synchronous calls
        _estimate("mock_128_host_f32", 128, 2000, 60000, 600000, call="sync", host=True),
        # one Gaussian mock of a wedge covariance study: a weighted object on every node, NGP, l <= 16
        _estimate("nodes_128_ngp_l16_f32", 128, 1000, 128 ** 3, 0, window=1, interlaced=False, compensated=False,
                  ell_max=16, catalog="nodes"),
        # uneven covariance mocks (128, 256 and 384 in turn) issued as one unit, one graph launch
        dict(name="batch_mocks_f32", kind="batch", mocks=6, box=2000.0, n_min=50001, n_max=800003, ell_max=4,
             precision=0, dk=0.01),
        # ordinary survey estimates, as a request loop issues them
        _estimate("survey_256_f32", 256, 2000, 400009, 4000037),
        _estimate("survey_384_f64", 384, 2000, 800011, 8000009, precision=1),
        # the benchmark estimate in both precision forms
        _estimate("survey_512_f32", 512, 2500, 1000000, 20000000),
        _estimate("survey_512_f64", 512, 2500, 1000000, 20000000, precision=1),
        # a radix-3 side that no shape table names, with more multipoles than usual
        _estimate("survey_432_l8_f32", 432, 2200, 700001, 7000003, ell_max=8, max_group=16),
        # the largest: fine wedges on 1024^3, fields in groups, wedges from the multipoles
        _estimate("wedges_1024_l8_f32", 1024, 3000, 4000000, 40000000, ell_max=8, max_group=12, mu_bins=5,
                  call="sync"),
        # fixed line of sight in a periodic box: (k, mu) cells
        dict(name="kmu_512_f32", kind="kmu", catalog="box", nmesh=512, box=2500.0, n_data=2000003, n_rand=0,
             window=3, interlaced=True, compensated=True, precision=0, dk=0.01, n_mu=10),
        # the 3D transform alone, forward and inverse, as a program that filters a density calls it
        dict(name="fft_512_f32", kind="fft", nmesh=512, precision=0),
    ]


def _fields(ell_max):
    return sum(2 * l + 1 for l in range(2, ell_max + 1, 2))


def draw(rng):
    """One more case of the same ranges."""
    nmesh = rng.choice(SIZES)
    precision = rng.choice((0, 0, 1))
    kind = rng.choice(("estimate",) * 8 + ("kmu", "fft"))
    if kind == "fft":
        return dict(kind="fft", nmesh=max(nmesh, 96), precision=precision)
    box = float(rng.randrange(900, 3000))
    cells = nmesh ** 3
    n_data = int(cells * 10.0 ** rng.uniform(-2.6, -1.0))
    n_data = max(3001, min(n_data, 2000003)) | 1
    window = rng.choice((1, 2, 3, 3))
    interlaced = rng.random() < 0.6
    compensated = rng.random() < 0.8
    dk = rng.choice((0.005, 0.01, 0.01, 0.02))
    while math.floor(math.pi * nmesh / box / dk) < 4:
        dk *= 0.5
    if kind == "kmu":
        while math.pi * nmesh / box / dk > 250:  # the call takes at most 3072 (k, mu) cells
            dk *= 2.0
        return dict(kind="kmu", catalog="box", nmesh=nmesh, box=box, n_data=n_data, n_rand=0, window=window,
                    interlaced=interlaced, compensated=compensated, precision=precision, dk=dk,
                    n_mu=rng.randrange(4, 11))
    ell_max = rng.choice((2, 4, 4, 4, 6, 8, 16))
    catalog = rng.choice(("survey", "survey", "survey", "box"))
    n_rand = 0 if catalog == "box" else int(n_data * rng.uniform(8.0, 20.0))
    es = 8 if precision else 4
    while (_fields(ell_max) + 3) * cells * (1 + precision) > LISTED_COST // 2:
        ell_max -= 2
    group = int(STATE_BYTES // (cells * es)) - 6
    c = _estimate("", nmesh, box, n_data, n_rand, window=window, interlaced=interlaced, compensated=compensated,
                  ell_max=ell_max, precision=precision, call=rng.choice(("sync", "async")), catalog=catalog,
                  host=n_data + n_rand < 3000000 and rng.random() < 0.2,
                  max_group=16 if group >= 16 and _fields(ell_max) > 16 and rng.random() < 0.5 else
                  (group if group < _fields(ell_max) else 0), dk=dk)
    if c["host"]:
        c["call"] = "sync"
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=torch.float64, device="cuda")


def _cone(g, n, box):
    """n points uniform in 0.4 L < r < 0.8 L within 30 degrees of +z around the observer."""
    r = (0.4 ** 3 + (0.8 ** 3 - 0.4 ** 3) * _rand(g, n)) ** (1.0 / 3.0) * box
    mu = 1.0 - (1.0 - math.cos(math.pi / 6)) * _rand(g, n)
    phi = 2.0 * math.pi * _rand(g, n)
    st = torch.sqrt(1.0 - mu * mu)
    return torch.stack((r * st * torch.cos(phi), r * st * torch.sin(phi), r * mu - 0.6 * box), dim=1)


def _clustered(g, n, box, points):
    """Half of the objects in clumps of about 20 with a spread of L/200, the rest unclustered."""
    pos = points(g, n, box)
    parents = points(g, max(8, n // 40), box)
    k = n // 2
    idx = torch.randint(parents.shape[0], (k,), generator=g, device="cuda")
    at = torch.randperm(n, generator=g, device="cuda")[:k]
    pos[at] = parents[idx] + (box / 200.0) * torch.randn(k, 3, generator=g, dtype=torch.float64, device="cuda")
    return pos.clamp_(-0.5 * box, 0.499999 * box)


def _uniform(g, n, box):
    return (_rand(g, n, 3) - 0.5) * box


def _catalogs(c, seed):
    """(data, randoms or None), each (positions, weights, nbar) on the GPU."""
    g = _gen(seed)
    box, nd, nr = c["box"], c["n_data"], c["n_rand"]
    if c["catalog"] == "nodes":
        n = c["nmesh"]
        x = torch.arange(n, dtype=torch.float64, device="cuda") * (box / n) - 0.5 * box
        pos = torch.stack(torch.meshgrid(x, x, x, indexing="ij"), dim=-1).reshape(-1, 3).contiguous()
        w = 1.0 + 0.3 * torch.randn(n ** 3, generator=g, dtype=torch.float64, device="cuda")
        return (pos, w, None), None
    if c["catalog"] == "box":
        return (_clustered(g, nd, box, _uniform), None, None), None
    volume = 2.0 * math.pi / 3.0 * (1.0 - math.cos(math.pi / 6)) * (0.8 ** 3 - 0.4 ** 3) * box ** 3
    nbar = nd / volume
    data = _clustered(g, nd, box, _cone)
    rand = _cone(g, nr, box)
    wd = 0.7 + 0.6 * _rand(g, nd)
    wr = 0.7 + 0.6 * _rand(g, nr)
    full = lambda n: torch.full((n,), nbar, dtype=torch.float64, device="cuda")  # noqa: E731
    return (data, wd, full(nd)), (rand, wr, full(nr))


def _observer(c):
    return (0.0, 0.0, -0.6 * c["box"])


def _edges(c, nmesh=None):
    kn = math.pi * (nmesh or c["nmesh"]) / c["box"]
    return np.arange(int(math.floor(kn / c["dk"])) + 1, dtype=np.float64) * c["dk"]


def _batch_mocks(c, seed):
    """The mocks' cases: sides 128, 256, 384 in turn, object counts log-uniform (fixed by position)."""
    out = []
    for i in range(c["mocks"]):
        f = (0.618034 * (i + 1)) % 1.0
        n = int(math.exp(math.log(c["n_min"]) + f * math.log(c["n_max"] / c["n_min"])))
        out.append(dict(_estimate("", (128, 256, 384)[i % 3], c["box"], n, 10 * n, ell_max=c["ell_max"],
                                  precision=c["precision"], dk=c["dk"]), seed=seed * 16 + i))
    return out


def _plan(c, **more):
    return Plan(c["nmesh"], c["box"], observer=_observer(c), window=c["window"], interlaced=c["interlaced"],
                compensated=c["compensated"], precision=c["precision"], **more)


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "fft":
        n = c["nmesh"]
        rdt, cdt = (torch.float64, torch.complex128) if c["precision"] else (torch.float32, torch.complex64)
        x = torch.randn(n, n, n, generator=_gen(seed), dtype=rdt, device="cuda")
        return dict(case=c, plan=Plan(n, 1000.0, precision=c["precision"], ell_max_hint=2, max_group=1), x=x,
                    half=torch.empty(n, n, n // 2, dtype=cdt, device="cuda"), back=torch.empty_like(x))
    if c["kind"] == "batch":
        batch, plans, keep = Batch(), {}, []
        mocks = _batch_mocks(c, seed)
        for m in mocks:
            # one plan and stream per mock: the estimates overlap on the device
            edges = _edges(m)
            p = _plan(m, ell_max_hint=m["ell_max"], stream=torch.cuda.Stream())
            p.prepare(m["ell_max"], edges, m["n_data"] + m["n_rand"])
            data, rand = _catalogs(m, m["seed"])
            plans[len(plans)] = p
            keep.append((data, rand))
            batch.add(p, data, rand)
        return dict(case=c, batch=batch, plans=plans, keep=keep)
    data, rand = _catalogs(c, seed)
    if c.get("host"):
        host = lambda cat: None if cat is None else tuple(None if a is None else a.cpu().numpy() for a in cat)  # noqa: E731
        data, rand = host(data), host(rand)
    edges = _edges(c)
    if c["kind"] == "kmu":
        return dict(case=c, plan=_plan(c, ell_max_hint=2, max_group=1, los=(0.0, 0.0, 1.0)), data=data, edges=edges,
                    mu=np.linspace(0.0, 1.0, c["n_mu"] + 1))
    plan = _plan(c, ell_max_hint=c["ell_max"], max_group=c["max_group"])
    if c["call"] == "async":
        plan.prepare(c["ell_max"], edges, c["n_data"] + c["n_rand"])
    return dict(case=c, plan=plan, data=data, rand=rand, edges=edges)


def _result(c, res):
    form = np.float64 if c["precision"] else np.float32
    return dict(poles=res["poles"].astype(form), k_mean=res["k_mean"], n_modes=res["n_modes"],
                norm_I=res["norm_I"], shot_noise=res["shot_noise"])


def run(state):
    c = state["case"]
    if c["kind"] == "fft":
        state["plan"].fft3d_forward(state["x"], state["half"])
        state["plan"].fft3d_inverse(state["half"], state["back"])
        return state["back"]
    if c["kind"] == "batch":
        b = state["batch"]
        b.run(use_graph=True)
        return [_result(c, b.result(i)) for i in range(c["mocks"])]
    plan = state["plan"]
    if c["kind"] == "kmu":
        plan.paint(state["data"])
        pk, nm = plan.kmu_global(state["edges"], state["mu"])
        return dict(pk=pk.astype(np.float64 if c["precision"] else np.float32), n_modes=nm)
    if c["call"] == "async":
        plan.enqueue(state["data"], state["rand"])
        res = plan.finish()
    else:
        plan.paint(state["data"], state["rand"])
        res = plan.compute_multipoles(c["ell_max"], state["edges"])
    out = _result(c, res)
    if c["mu_bins"]:
        w = wedges(res["poles"], c["ell_max"], nonuniform_mu_edges(c["ell_max"]))
        out["wedges"] = w.astype(out["poles"].dtype)
    return out


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
def _estimate_work(c, fields):
    """Catalog objects (40 bytes) read once; transforms of real meshes (2.5 N^3 log2 N^3
    flops each), two weights per field and cell, the assignment taps of every object."""
    n3 = float(c["nmesh"]) ** 3
    meshes = 2 if c["interlaced"] else 1
    transforms = fields + meshes + (1 if c["interlaced"] or c["compensated"] else 0)
    objects = c["n_data"] + c["n_rand"]
    per = 24.0 + (0.0 if c["catalog"] == "box" else 8.0 if c["catalog"] == "nodes" else 16.0)
    return dict(bytes=per * objects, flops=transforms * 2.5 * n3 * math.log2(n3) + 6.0 * fields * n3 +
                2.0 * meshes * c["window"] ** 3 * objects)


def work(case):
    if case["kind"] == "fft":
        n3 = float(case["nmesh"]) ** 3
        return dict(bytes=2.0 * n3 * (8 if case["precision"] else 4), flops=2 * 2.5 * n3 * math.log2(n3))
    if case["kind"] == "batch":
        parts = [_estimate_work(m, _fields(m["ell_max"])) for m in _batch_mocks(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    return _estimate_work(case, 0 if case["kind"] == "kmu" else _fields(case["ell_max"]))


# ---------------------------------------------------------------------------------------------
# the same results in 64 bits with plain torch
# ---------------------------------------------------------------------------------------------
def _taps(u, window):
    if window == 2:
        c = torch.floor(u)
        d = u - c
        return c.long(), (1.0 - d, d)
    c = torch.floor(u + 0.5)
    d = u - c
    if window == 1:
        return c.long(), (torch.ones_like(d),)
    return c.long() - 1, (0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2)


def _paint(mesh, pos, w, c, shift, factor):
    n = c["nmesh"]
    for i in range(0, pos.shape[0], 4000000):
        u = (pos[i:i + 4000000] + 0.5 * c["box"]) * (n / c["box"]) + shift
        wt = torch.full((u.shape[0],), 1.0, dtype=torch.float64, device="cuda") if w is None else w[i:i + 4000000]
        wt = wt * factor
        base, t = _taps(u, c["window"])
        for a in range(len(t)):
            ia = (base[:, 0] + a) % n
            for b in range(len(t)):
                ib = ia * n + (base[:, 1] + b) % n
                wab = wt * t[a][:, 0] * t[b][:, 1]
                for e in range(len(t)):
                    mesh.index_add_(0, ib * n + (base[:, 2] + e) % n, wab * t[e][:, 2])


def _freq(n):
    f = torch.arange(n, dtype=torch.float64, device="cuda")
    return torch.where(f < n / 2, f, f - n)


def _combined(c, data, rand, alpha):
    """C on kz < N/2 and the field that is harmonically weighted."""
    n, nh = c["nmesh"], c["nmesh"] // 2
    f = _freq(n)
    half = f[:nh]
    total = None
    for shift in ((0.0, 0.5) if c["interlaced"] else (0.0,)):
        mesh = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
        _paint(mesh, data[0], data[1], c, shift, 1.0)
        if rand is not None:
            _paint(mesh, rand[0], rand[1], c, shift, -alpha)
        mesh = mesh.view(n, n, n)
        s = torch.fft.rfftn(mesh)[:, :, :nh]
        if shift:
            for x in range(n):
                ph = math.pi / n * (f[x] + f[:, None] + half[None, :])
                total[x] = 0.5 * (total[x] + torch.polar(torch.ones_like(ph), ph) * s[x])
        else:
            total = s.clone()
        del s
    x = math.pi * f / n
    if c["compensated"]:
        if c["interlaced"]:
            wc = torch.where(f == 0, torch.ones_like(x), torch.sin(x) / torch.where(f == 0, torch.ones_like(x), x)) ** c["window"]
        else:
            s2 = torch.sin(x) ** 2
            wc = torch.sqrt({1: torch.ones_like(s2), 2: 1.0 - 2.0 / 3.0 * s2, 3: 1.0 - s2 + 2.0 / 15.0 * s2 * s2}[c["window"]])
        for i in range(n):
            total[i] /= wc[i] * wc[:, None] * wc[None, :nh]
    total[nh] = 0
    total[:, nh] = 0
    if not (c["interlaced"] or c["compensated"]):
        return total, mesh
    del mesh
    full = torch.zeros(n, n, nh + 1, dtype=torch.complex128, device="cuda")
    full[:, :, :nh] = total
    return total, torch.fft.irfftn(full, s=(n, n, n), dim=(0, 1, 2))


def _ylm(l, m, ux, uy, uz):
    am = abs(m)
    cr, ci = torch.ones_like(uz), torch.zeros_like(uz)
    for _ in range(am):
        cr, ci = cr * ux - ci * uy, cr * uy + ci * ux
    q = 1.0
    for j in range(1, am + 1):
        q *= (2.0 * j - 1.0) / (2.0 * j)
    top = math.sqrt((2.0 * am + 1.0) * q / (4.0 * math.pi) * (2.0 if am else 1.0))
    q0, q1 = torch.zeros_like(uz), torch.full_like(uz, top)
    for j in range(am + 1, l + 1):
        a = math.sqrt((4.0 * j * j - 1.0) / (j * j - am * am))
        b = math.sqrt(((j - 1.0) ** 2 - am * am) * (2.0 * j + 1.0) / ((2.0 * j - 3.0) * (j * j - am * am))) if j > am + 1 else 0.0
        q0, q1 = q1, a * uz * q1 - b * q0
    return q1 * (ci if m < 0 else cr)


def _slabs(n):
    step = max(1, int(2.0e7 // (n * n)))
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _unit(x, y, z):
    r = torch.sqrt(x * x + y * y + z * z)
    inv = torch.where(r > 0, 1.0 / torch.where(r > 0, r, torch.ones_like(r)), torch.zeros_like(r))
    return x * inv, y * inv, z * inv


def _node_units(c, s):
    n, o = c["nmesh"], _observer(c)
    x = torch.arange(n, dtype=torch.float64, device="cuda") * (c["box"] / n) - 0.5 * c["box"]
    return _unit((x[s] - o[0])[:, None, None], (x - o[1])[None, :, None], (x - o[2])[None, None, :])


def _mode_vec(c, s):
    f = _freq(c["nmesh"])
    return f[s][:, None, None], f[None, :, None], f[None, None, :c["nmesh"] // 2]


def _thresholds(edges, box):
    return torch.as_tensor(np.ceil(((edges * box) / (2.0 * math.pi)) ** 2), dtype=torch.float64, device="cuda")


def _bins(c, s, thr):
    """Bin of every mode of a slab (the last index collects the modes of no bin), weights, |n|^2."""
    n, nb = c["nmesh"], thr.numel() - 1
    x, y, z = _mode_vec(c, s)
    n2 = x * x + y * y + z * z
    idx = torch.bucketize(n2, thr, right=True) - 1
    bad = (idx < 0) | (idx >= nb) | (n2 == 0) | (x == -(n // 2)) | (y == -(n // 2))
    w = torch.where(z == 0, 1.0, 2.0).to(torch.float64).expand(n2.shape)
    return torch.where(bad, torch.full_like(idx, nb), idx), w, n2


def _sum(idx, val, nb):
    return torch.bincount(idx.reshape(-1), weights=val.reshape(-1), minlength=nb + 1)[:nb]


def _scalars(c, data, rand):
    sq = lambda cat: float((torch.ones_like(cat[0][:, 0]) if cat[1] is None else cat[1] ** 2).sum())  # noqa: E731
    if rand is None:
        nbar = data[0].shape[0] / c["box"] ** 3
        norm = nbar * sq(data)
        return 0.0, norm, sq(data) / norm
    alpha = data[0].shape[0] / rand[0].shape[0]
    norm = alpha * float((rand[1] ** 2 * rand[2]).sum())
    return alpha, norm, (sq(data) + alpha ** 2 * sq(rand)) / norm


def _exact_estimate(c, seed):
    data, rand = _catalogs(c, seed)
    alpha, norm, shot = _scalars(c, data, rand)
    cf, dc = _combined(c, data, rand, alpha)
    n, nh = c["nmesh"], c["nmesh"] // 2
    edges = _edges(c)
    thr = _thresholds(edges, c["box"])
    nb = thr.numel() - 1
    zero = lambda: torch.zeros(nb, dtype=torch.float64, device="cuda")  # noqa: E731
    count, ksum, poles = zero(), zero(), []
    for ell in range(0, c["ell_max"] + 1, 2):
        if ell == 0:
            acc = cf
        else:
            acc = torch.zeros_like(cf)
            weighted = torch.empty_like(dc)
            for m in range(-ell, ell + 1):
                for s in _slabs(n):
                    weighted[s] = dc[s] * _ylm(ell, m, *_node_units(c, s))
                b = torch.fft.rfftn(weighted)
                for s in _slabs(n):
                    acc[s] += _ylm(ell, m, *_unit(*_mode_vec(c, s))) * b[s][:, :, :nh]
                del b
            acc *= 4.0 * math.pi / (2 * ell + 1)
        q = zero()
        for s in _slabs(n):
            idx, w, n2 = _bins(c, s, thr)
            q += _sum(idx, w * (cf[s] * acc[s].conj()).real, nb)
            if ell == 0:
                count += _sum(idx, w, nb)
                ksum += _sum(idx, w * torch.sqrt(n2) * (2.0 * math.pi / c["box"]), nb)
        poles.append((2 * ell + 1) * q / (norm * count) - (shot if ell == 0 else 0.0))
    poles = torch.stack(poles).cpu().numpy()
    out = dict(poles=poles, k_mean=(ksum / count).cpu().numpy(), n_modes=None, norm_I=norm, shot_noise=shot)
    if c["mu_bins"]:
        out["wedges"] = _exact_wedges(poles, nonuniform_edges(c["ell_max"]))
    return out


def _legendre(l, x):
    return np.polynomial.legendre.legval(x, [0.0] * l + [1.0])


def nonuniform_edges(ell_max):
    """mu_0 = 0, then the edges at which every wedge but the first integrates L_{ell_max+1}(mu)/mu
    to zero: roots of its antiderivative's difference from the value at 1."""
    c = np.polynomial.legendre.leg2poly([0.0] * (ell_max + 1) + [1.0])
    anti = np.polynomial.Polynomial(np.concatenate(([0.0], c[1:] / np.arange(1.0, len(c)))))
    f = lambda x: anti(x) - anti(1.0)  # noqa: E731
    # between consecutive extrema (the roots of L_{ell_max+1}) lies one crossing
    roots = np.sort(np.polynomial.legendre.legroots([0.0] * (ell_max + 1) + [1.0]))
    roots = np.concatenate(([1e-9], roots[roots > 1e-9]))
    edges = [0.0]
    for lo, hi in zip(roots[:-1], roots[1:]):
        if f(lo) * f(hi) < 0:
            for _ in range(200):
                mid = 0.5 * (lo + hi)
                lo, hi = (mid, hi) if f(lo) * f(mid) > 0 else (lo, mid)
            edges.append(0.5 * (lo + hi))
    return np.array(edges + [1.0])


def _exact_wedges(poles, mu):
    out = np.zeros((poles.shape[1], len(mu) - 1))
    for i in range(poles.shape[0]):
        l = 2 * i
        for j in range(len(mu) - 1):
            a, b = mu[j], mu[j + 1]
            up, dn = l + 1, l - 1
            lbar = 1.0 if l == 0 else ((_legendre(up, b) - _legendre(dn, b)) - (_legendre(up, a) - _legendre(dn, a))) / ((2 * l + 1) * (b - a))
            out[:, j] += poles[i] * lbar
    return out


def _exact_kmu(c, seed):
    data, _ = _catalogs(c, seed)
    alpha, norm, shot = _scalars(c, data, None)
    cf, _ = _combined(c, data, None, alpha)
    n, nmu = c["nmesh"], c["n_mu"]
    thr = _thresholds(_edges(c), c["box"])
    nb = thr.numel() - 1
    mue = torch.as_tensor(np.linspace(0.0, 1.0, nmu + 1), device="cuda")
    cnt = torch.zeros(nb * nmu, dtype=torch.float64, device="cuda")
    tot = torch.zeros_like(cnt)
    for s in _slabs(n):
        idx, w, n2 = _bins(c, s, thr)
        z = _mode_vec(c, s)[2].expand(n2.shape)
        mu = z.abs() / torch.sqrt(n2)
        mb = (torch.bucketize(mu, mue, right=True) - 1).clamp(0, nmu - 1)
        cell = torch.where(idx == nb, torch.full_like(idx, nb * nmu), idx * nmu + mb)
        cnt += _sum(cell, w, nb * nmu)
        tot += _sum(cell, w * (cf[s].real ** 2 + cf[s].imag ** 2), nb * nmu)
    return dict(pk=(tot / (norm * cnt) - shot).view(nb, nmu).cpu().numpy(), n_modes=None)


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "fft":
        n = c["nmesh"]
        rdt = torch.float64 if c["precision"] else torch.float32
        x = torch.randn(n, n, n, generator=_gen(seed), dtype=rdt, device="cuda").double()
        s = torch.fft.rfftn(x)
        s[:, :, n // 2] = 0
        return torch.fft.irfftn(s, s=(n, n, n), dim=(0, 1, 2))
    if c["kind"] == "batch":
        return [_exact_estimate(m, m["seed"]) for m in _batch_mocks(c, seed)]
    return _exact_kmu(c, seed) if c["kind"] == "kmu" else _exact_estimate(c, seed)
