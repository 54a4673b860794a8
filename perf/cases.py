"""The pair counts a program asks of this package, as cases to be timed.

A case is a dict of plain values.  ``listed()`` names the fixed ones,
``draw(rng)`` gives one more of the same ranges, ``prepare(case, seed)`` makes
the inputs, ``run(state)`` is one call of the package's public entry point,
``work(case)`` the bytes and operations such a call cannot do without and
``exact(case, seed)`` the floating outputs in plain torch float64.

Inputs follow the package's synthetic catalogues: boxes with half of the
points uniform and half in Gaussian blobs (width 2, 200 points of the box per
blob), a 30-degree cap with 0.1-degree blobs, a 10-degree cone of on-sky
galaxies between distances 500 and 1500.  They are drawn on the GPU from the
seed alone.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1911_03545_amd as pc

_DEV = "cuda:0"
_COUNTER = None
_SIGMA = 2.0
_CAP_DEG = 30.0
_CONE_DEG, _CONE_MIN, _CONE_MAX = 10.0, 500.0, 1500.0


def _counter():
    """The one library handle that a program keeps for all its calls."""
    global _COUNTER
    if _COUNTER is None:
        _COUNTER = pc.PairCounter(0)
    return _COUNTER


def _case(name, stat, n, **more):
    c = {"name": name, "stat": stat, "n": n, "n2": 0, "box": 0.0, "lo": 0.1, "hi": 25.0,
         "nb": 20, "pimax": 40.0, "npi": 40, "prec": "fp32", "f32": False, "host": False,
         "weights": "", "ravg": False, "ncat": 1, "sizes_seed": 0}
    c.update(more)
    return c


def listed():
    return [
        # a small simulation box, as in a notebook or a fit's inner loop: the
        # call is latency and launches
        _case("r_small", "r", 10_000, box=100.0, hi=10.0),
        # a script on NumPy arrays with the default precision: float32
        # columns in host memory, an odd number of points
        _case("r_host_f64", "r", 100_003, box=210.0, hi=20.0, nb=14, prec="fp64", f32=True,
              host=True),
        # xi(r) of a galaxy mock: the benchmark's catalogue, both precisions
        _case("r_box_f32", "r", 1_000_000, box=420.0),
        _case("r_box_f64", "r", 1_000_000, box=420.0, prec="fp64"),
        # wp(rp) of the same mock
        _case("rppi_box_f32", "rppi", 1_000_000, box=420.0),
        # weighted xi(r) of a large halo catalogue
        _case("r_weighted_f32", "r", 4_000_000, box=1100.0, hi=50.0, nb=25, weights="product"),
        # weighted wp(rp) with the mean separation of every bin, in binary64
        _case("rppi_ravg_f64", "rppi", 300_007, box=281.0, prec="fp64", weights="product",
              ravg=True),
        # xi(r) of galaxies against randoms without a periodic box (the DR
        # term of a survey estimator), weighted by the sum of the weights
        _case("r_cross_open_f32", "r", 150_001, n2=600_011, box=0.0, weights="sum"),
        # w(theta) of a wide survey: DD on a cap
        _case("theta_dd_f32", "theta", 2_000_000, lo=0.01, hi=10.0),
        # its DR term from host arrays, in binary64
        _case("theta_dr_f64", "theta", 200_001, n2=500_009, lo=0.01, hi=5.0, nb=15, prec="fp64",
              host=True),
        # wp(rp) of an on-sky galaxy survey
        _case("mocks_f64", "mocks", 1_000_000, prec="fp64"),
        # wp(rp) of many mock catalogues of a fit in one call: sizes between
        # n / 10 and n
        _case("batch_f32", "batch", 2_000_000, box=1000.0, ncat=48, sizes_seed=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the listed ones' ranges, of no greater cost."""
    stat = rng.choice(["r", "r", "rppi", "rppi", "cross", "theta", "mocks", "batch"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    more = {"prec": prec, "nb": rng.randint(8, 30), "f32": rng.random() < 0.3}
    if stat in ("r", "rppi", "cross"):
        n = _log_int(rng, 3e3, 1.5e6)
        density = math.exp(rng.uniform(math.log(2e-3), math.log(1.4e-2)))
        box = round((n / density) ** (1.0 / 3.0), 2)
        most = min(25.0, 0.3 * box)
        hi = round(rng.uniform(0.4 * most, most), 2)
        pimax = round(min(40.0, 0.3 * box))
        more.update(box=box, hi=hi, pimax=float(pimax), npi=max(1, int(pimax)),
                    weights=rng.choice(["", "", "product", "sum"]),
                    host=rng.random() < 0.25)
        more["ravg"] = rng.random() < 0.2
        if stat == "cross":
            stat = rng.choice(["r", "rppi"])
            more.update(n2=_log_int(rng, max(3e3, n / 5), min(1.5e6, 5.0 * n)),
                        box=rng.choice([0.0, box]))
            if more["box"] == 0.0:
                more["host"] = False
        return {k: v for k, v in _case("", stat, n, **more).items() if k != "name"}
    if stat == "theta":
        n = _log_int(rng, 1e4, 1e6)
        more.update(lo=0.01, hi=round(rng.uniform(1.0, 10.0), 2), host=rng.random() < 0.5,
                    n2=rng.choice([0, _log_int(rng, 1e4, 6e5)]))
    elif stat == "mocks":
        n = _log_int(rng, 1e4, 1e6)
        more.update(hi=round(rng.uniform(8.0, 25.0), 2), host=rng.random() < 0.3)
    else:
        n = _log_int(rng, 5e3, 1.5e6)
        density = math.exp(rng.uniform(math.log(5e-4), math.log(5e-3)))
        box = round((n / density) ** (1.0 / 3.0), 2)
        pimax = round(min(40.0, 0.3 * box))
        more.update(box=box, hi=round(min(25.0, 0.3 * box), 2), pimax=float(pimax),
                    npi=max(1, int(pimax)), ncat=rng.randint(2, 32),
                    sizes_seed=rng.randint(1, 10_000), f32=False)
    return {k: v for k, v in _case("", stat, n, **more).items() if k != "name"}


# ---- inputs ---------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=_DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=_DEV, dtype=torch.float64)


def _box_points(g, n, side):
    """Half uniform, half in blobs, wrapped into the box, in random order."""
    n_cl = n // 2
    blobs = max(1, n // 200)
    centres = _rand(g, 3, blobs) * side
    owner = torch.randint(blobs, (n_cl,), generator=g, device=_DEV)
    cl = torch.remainder(centres[:, owner] + _SIGMA * _randn(g, 3, n_cl), side)
    p = torch.cat([_rand(g, 3, n - n_cl) * side, cl], dim=1)
    return p[:, torch.randperm(n, generator=g, device=_DEV)].clamp_(0.0, side)


def _directions(g, n, radius_deg):
    """Unit vectors uniform on a cap around (RA, DEC) = (0, 30) degrees."""
    ct = 1.0 - _rand(g, n) * (1.0 - math.cos(math.radians(radius_deg)))
    st = torch.sqrt((1.0 - ct * ct).clamp_min(0.0))
    ph = 2.0 * math.pi * _rand(g, n)
    c, s = math.cos(math.radians(30.0)), math.sin(math.radians(30.0))
    e, nn = st * torch.sin(ph), st * torch.cos(ph)
    return torch.stack([c * ct - s * nn, e, s * ct + c * nn])


def _radec(v):
    ra = torch.rad2deg(torch.atan2(v[1], v[0]))
    ra = torch.where(ra < 0.0, ra + 360.0, ra).clamp_(0.0, 360.0)
    return ra, torch.rad2deg(torch.asin(v[2].clamp(-1.0, 1.0)))


def _cap(g, n, clustered):
    v = _directions(g, n, _CAP_DEG)
    if clustered:
        n_cl = n // 2
        blobs = max(1, n // 200)
        centres = _directions(g, blobs, _CAP_DEG - 0.5)
        owner = torch.randint(blobs, (n_cl,), generator=g, device=_DEV)
        cl = centres[:, owner] + math.radians(0.1) * _randn(g, 3, n_cl)
        v[:, :n_cl] = cl / cl.norm(dim=0)
        v = v[:, torch.randperm(n, generator=g, device=_DEV)]
    return _radec(v)


def _cone(g, n):
    d = (_CONE_MIN ** 3 + _rand(g, n) * (_CONE_MAX ** 3 - _CONE_MIN ** 3)) ** (1.0 / 3.0)
    p = _directions(g, n, _CONE_DEG) * d
    n_cl = n // 2
    blobs = max(1, n // 200)
    dc = (_CONE_MIN ** 3 + _rand(g, blobs) * (_CONE_MAX ** 3 - _CONE_MIN ** 3)) ** (1.0 / 3.0)
    centres = _directions(g, blobs, _CONE_DEG) * dc
    owner = torch.randint(blobs, (n_cl,), generator=g, device=_DEV)
    p[:, :n_cl] = centres[:, owner] + _SIGMA * _randn(g, 3, n_cl)
    p = p[:, torch.randperm(n, generator=g, device=_DEV)]
    d = p.norm(dim=0)
    ra, dec = _radec(p / d)
    return ra, dec, d


def _columns(case, cols):
    """The columns as the caller holds them: float32 or float64, on the GPU
    or as NumPy arrays."""
    out = []
    for c in cols:
        c = c.to(torch.float32) if case["f32"] else c
        c = c.contiguous()
        if case["f32"] and case["box"] > 0.0:
            c = torch.minimum(c, torch.tensor(_f32_below(case["box"]), device=_DEV))
        out.append(c.cpu().numpy() if case["host"] else c)
    return tuple(out)


def _f32_below(x):
    f = np.float32(x)
    return float(f if float(f) <= x else np.nextafter(f, np.float32(0.0)))


def _weights(case, g, n):
    w = (0.5 + _rand(g, n)).to(torch.float32)
    return w.cpu().numpy() if case["host"] else w


def _sizes(case):
    r = random.Random(case["sizes_seed"])
    return [r.randint(max(1, case["n"] // 10), case["n"]) for _ in range(case["ncat"])]


def _edges(case):
    return np.logspace(math.log10(case["lo"]), math.log10(case["hi"]), case["nb"] + 1)


def _inputs(case, seed):
    g = _gen(seed)
    s = {"case": case, "edges": _edges(case), "d1": None, "d2": None, "w1": None, "w2": None}
    stat, n, n2 = case["stat"], case["n"], case["n2"]
    if stat in ("r", "rppi"):
        # without a periodic box both catalogues fill one of the mock's density
        side = case["box"] or (max(n, n2) / 0.0135) ** (1.0 / 3.0)
        s["d1"] = _columns(case, _box_points(g, n, side))
        if n2:
            s["d2"] = _columns(case, _rand(g, 3, n2) * side)
        if case["weights"]:
            s["w1"] = _weights(case, g, n)
            s["w2"] = _weights(case, g, n2) if n2 else None
    elif stat == "theta":
        s["d1"] = _columns(case, _cap(g, n, True))
        if n2:
            s["d2"] = _columns(case, _cap(g, n2, False))
    elif stat == "mocks":
        s["d1"] = _columns(case, _cone(g, n))
    else:
        s["d1"] = [_columns(case, _box_points(g, m, case["box"])) for m in _sizes(case)]
    return s


def prepare(case, seed):
    _counter()
    return _inputs(case, seed)


def run(state):
    c, k = state["case"], _counter()
    stat = c["stat"]
    kind = c["weights"] or None
    if stat == "r":
        return k.count_r(state["d1"], state["d2"], state["edges"], c["box"], c["prec"],
                         w1=state["w1"], w2=state["w2"], weight_type=kind, ravg=c["ravg"])
    if stat == "rppi":
        return k.count_rppi(state["d1"], state["d2"], state["edges"], c["pimax"], c["npi"],
                            c["box"], c["prec"], w1=state["w1"], w2=state["w2"],
                            weight_type=kind, ravg=c["ravg"])
    if stat == "theta":
        d2 = state["d2"] or (None, None)
        return k.count_theta(state["d1"][0], state["d1"][1], d2[0], d2[1], state["edges"],
                             c["prec"])
    if stat == "mocks":
        return k.count_rppi_mocks(state["d1"], None, state["edges"], c["pimax"], c["npi"],
                                  c["prec"])
    return k.count_rppi_batch(state["d1"], state["edges"], c["pimax"], c["npi"], c["box"],
                              c["prec"])


# ---- what a call cannot do without ------------------------------------------
def _in_range(case, n, n2, box):
    """Expected unordered (cross: all) pairs in range."""
    stat, hi = case["stat"], case["hi"]
    if stat == "r":
        f = 4.0 / 3.0 * math.pi * hi ** 3 / box ** 3
    elif stat in ("rppi", "batch"):
        f = math.pi * hi * hi * 2.0 * case["pimax"] / box ** 3
    elif stat == "theta":
        f = (1.0 - math.cos(math.radians(hi))) / (1.0 - math.cos(math.radians(_CAP_DEG)))
    else:
        cone = 2.0 * math.pi * (1.0 - math.cos(math.radians(_CONE_DEG))) / 3.0 * (
            _CONE_MAX ** 3 - _CONE_MIN ** 3)
        f = math.pi * hi * hi * 2.0 * case["pimax"] / cone
    f = min(f, 1.0)
    if n2:
        return float(n) * n2 * f
    # the uniform expectation, and about 100 points of one blob in range
    return 0.5 * n * n * f + 0.5 * (n / 2) * 100.0


def work(case):
    """Each column read once and each output written once; eight operations
    (three differences, three squares, two sums) for every pair in range."""
    stat = case["stat"]
    item = 4 if case["f32"] else 8
    cols = 2 if stat == "theta" else 3
    sizes = _sizes(case) if stat == "batch" else [case["n"]]
    n, n2 = sum(sizes), case["n2"]
    box = case["box"] or (max(case["n"], n2) / 0.0135) ** (1.0 / 3.0)
    bins = case["nb"] * (case["npi"] if stat in ("rppi", "mocks", "batch") else 1) * len(sizes)
    outs = 1 + (1 if case["weights"] else 0) + (1 if case["ravg"] else 0)
    pairs = sum(_in_range(case, m, n2, box) for m in sizes)
    return {"bytes": float((n + n2) * (cols * item + (4 if case["weights"] else 0)) +
                           8 * bins * outs),
            "flops": 8.0 * pairs}


# ---- the floating outputs in plain float64 ----------------------------------
_EXACT_MOST = 1.5e11   # ordered candidate pairs (about 20 seconds)


def exact(case, seed):
    """(None, weight sums, mean separations) of the r and (rp, pi) counts by
    plain float64 torch over cells of at least the reach; None where a case
    has no floating outputs or too many pairs.  The counts are whole numbers
    and are compared as they are."""
    if case["stat"] not in ("r", "rppi") or not (case["weights"] or case["ravg"]):
        return None
    s = _inputs(case, seed)
    rp = case["stat"] == "rppi"
    box = case["box"]

    def on_gpu(cols):
        return [torch.as_tensor(c).to(_DEV).to(torch.float64) for c in cols]

    p = torch.stack(on_gpu(s["d1"]))
    q = p if s["d2"] is None else torch.stack(on_gpu(s["d2"]))
    one = lambda m: torch.ones(m, device=_DEV, dtype=torch.float64)  # noqa: E731
    wp = one(p.shape[1]) if s["w1"] is None else on_gpu([s["w1"]])[0]
    wq = wp if s["d2"] is None else (one(q.shape[1]) if s["w2"] is None
                                     else on_gpu([s["w2"]])[0])
    auto = s["d2"] is None
    side = box or float(torch.maximum(p.max(), q.max())) * (1.0 + 1e-12)
    reach = [case["hi"], case["hi"], case["pimax"] if rp else case["hi"]]
    nc = [max(1, int(side / (r * (1.0 + 1e-9)))) for r in reach]
    if p.shape[1] * q.shape[1] * 27.0 / (nc[0] * nc[1] * nc[2]) > _EXACT_MOST:
        return None

    def by_cell(v):
        i = [(v[a] * (nc[a] / side)).long().clamp_(0, nc[a] - 1) for a in range(3)]
        cell = (i[0] * nc[1] + i[1]) * nc[2] + i[2]
        order = torch.argsort(cell, stable=True)
        cnt = torch.bincount(cell, minlength=nc[0] * nc[1] * nc[2])
        start = torch.cat([torch.zeros(1, dtype=torch.long, device=_DEV), cnt.cumsum(0)])
        return order, start.tolist()

    op, sp = by_cell(p)
    p, wp = p[:, op].contiguous(), wp[op]
    oq, sq = (op, sp) if auto else by_cell(q)
    q, wq = (p, wp) if auto else (q[:, oq].contiguous(), wq[oq])
    e = torch.from_numpy(_edges(case)).to(_DEV)
    e2 = e * e
    npi = case["npi"] if rp else 1
    dpi = case["pimax"] / npi
    qe = torch.tensor([k * dpi for k in range(npi)] + [case["pimax"]], device=_DEV,
                      dtype=torch.float64)
    nbt = case["nb"] * npi
    wsum = torch.zeros(nbt, device=_DEV, dtype=torch.float64)
    rsum = torch.zeros(nbt, device=_DEV, dtype=torch.float64)

    def neighbours(a, i):
        if box > 0.0:
            return sorted({(i + d) % nc[a] for d in (-1, 0, 1)})
        return [j for j in (i - 1, i, i + 1) if 0 <= j < nc[a]]

    def gap(u, v):
        d = (u[:, None] - v[None, :]).abs_()
        return torch.minimum(d, box - d) if box > 0.0 else d

    for ix in range(nc[0]):
        for iy in range(nc[1]):
            for iz in range(nc[2]):
                c = (ix * nc[1] + iy) * nc[2] + iz
                a0, a1 = sp[c], sp[c + 1]
                if a0 == a1:
                    continue
                parts = [(sq[d], sq[d + 1])
                         for jx in neighbours(0, ix) for jy in neighbours(1, iy)
                         for jz in neighbours(2, iz)
                         for d in [(jx * nc[1] + jy) * nc[2] + jz]]
                v = torch.cat([q[:, b0:b1] for b0, b1 in parts], dim=1)
                w = torch.cat([wq[b0:b1] for b0, b1 in parts])
                step = max(1, int(4e7) // max(1, v.shape[1]))
                for b0 in range(a0, a1, step):
                    b1 = min(a1, b0 + step)
                    dx, dy = gap(p[0, b0:b1], v[0]), gap(p[1, b0:b1], v[1])
                    dz = gap(p[2, b0:b1], v[2])
                    sep = dx * dx + dy * dy
                    if not rp:
                        sep = sep + dz * dz
                    ok = (sep >= e2[0]) & (sep < e2[-1])
                    if rp:
                        ok &= dz < case["pimax"]
                    at = ok.nonzero(as_tuple=True)
                    sep = sep[at]
                    k = torch.bucketize(sep, e2, right=True) - 1
                    if rp:
                        k = k * npi + (torch.bucketize(dz[at], qe, right=True) - 1)
                    wi, wj = wp[b0:b1][at[0]], w[at[1]]
                    ww = wi + wj if case["weights"] == "sum" else wi * wj
                    wsum += torch.bincount(k, weights=ww, minlength=nbt)
                    if case["ravg"]:
                        rsum += torch.bincount(k, weights=ww * sep.sqrt(), minlength=nbt)
    shape = (case["nb"], npi) if rp else (case["nb"],)
    out = [None, wsum.reshape(shape) if case["weights"] else None]
    if case["ravg"]:
        out.append(torch.where(wsum != 0.0, rsum / wsum, torch.zeros_like(rsum)).reshape(shape))
    return tuple(out)
