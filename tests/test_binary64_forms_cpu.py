"""Error bounds of the binary64 forms in fewer operations, checked on the CPU with
the sweep's own arithmetic (fused multiply-adds rounded once, from exact
rationals): the expanded DD(r) within cf_expand64_bound of the definition, the
on-sky form within cf_mocks_bounds -- for random pairs, pairs at the largest
coordinates, wrapped pairs, coincident ones and pairs on the edges -- and the
limits at which either form is given up.  Each check also says how much of the
bound it meets, so that a bound some times smaller would be caught."""
from fractions import Fraction

import numpy as np
import pytest

import paper_1911_03545_amd as pc
import synth


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def expanded(p, q, D, c):
    """(s, definition) of one pair: p shifted by D against q, scale c; s unscaled."""
    c2 = c * c
    a = [x + d for x, d in zip(p, D)]
    A = ((a[0] * a[0] + a[1] * a[1]) + a[2] * a[2]) * c2
    t = A + ((q[0] * q[0] + q[1] * q[1]) + q[2] * q[2]) * c2
    f = -2.0 * c2
    for k in range(3):
        t = fma(f * a[k], q[k], t)
    d = [(x - y) + s for x, y, s in zip(p, q, D)]
    s = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
    return t, s


def pairs_near(rng, n, lo, hi, reach, edges):
    p = rng.uniform(lo, hi, (n, 3))
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    r = np.where(rng.random(n) < 0.5, rng.choice(edges, n), reach * rng.random(n))
    q = np.clip(p + u * r[:, None], lo, hi)
    q[: n // 16] = p[: n // 16]
    return p, q


@pytest.mark.parametrize("shift,box", [(0.0, 100.0), (0.0, 0.0), (1e3, 0.0), (9e3, 0.0)])
def test_expanded_r_within_its_bound(shift, box):
    edges = np.r_[0.0, np.logspace(-1.0, 1.0, 12)]
    rng = synth.rng_for(int(shift) + int(box))
    mag = 15.0 * box * box if box else 6.0 * (shift + 100.0) ** 2
    bound, c = pc.expand64_bound(edges, mag)
    assert bound > 0.0 and bound == 32.0 * 2.0 ** -53 * mag
    p, q = pairs_near(rng, 6000, shift, shift + 100.0, 10.0, edges[1:])
    D = np.zeros((len(p), 3))
    if box:
        D = box * rng.integers(-1, 2, p.shape)
        q = np.clip(q + D, 0.0, box) if box else q
    worst = 0.0
    for k in range(len(p)):
        t, s = expanded(p[k].tolist(), q[k].tolist(), D[k].tolist(), c)
        err = abs(Fraction(t) / (Fraction(c) * Fraction(c)) - Fraction(s))
        worst = max(worst, float(err) / bound)
    print("expanded r: largest share of the bound", worst)
    # (mag is the sum at its largest: wrapped pairs reach a third of it at most)
    assert 2.0 ** -8 < worst < 0.5


def test_expanded_r_limits():
    """Taken while the bound is at most 2^-12 of the smallest nonzero squared edge
    and 2^-18 of the largest, for byte tables; the scaled top lies in the key."""
    u = 32.0 * 2.0 ** -53
    for edges in (np.r_[0.0, 0.5, 4.0], np.r_[0.01, 9.0], np.r_[0.0, 3.0]):
        e = edges[edges > 0]
        most = min(2.0 ** -12 * e[0] ** 2, 2.0 ** -18 * e[-1] ** 2) / u
        assert pc.expand64_bound(edges, most * (1 + 1e-12)) == (0.0, 0.0)
        d, c = pc.expand64_bound(edges, most * (1 - 1e-12))
        assert d > 0.0 and (e[-1] ** 2 + d) * c * c < 32766.0 / 32767.0
        assert d * c * c < 0.5 / 32767   # (a sum below zero still has the key 0)
    assert pc.expand64_bound(np.linspace(0.0, 1.0, 126), 1.0)[0] > 0.0
    assert pc.expand64_bound(np.linspace(0.0, 1.0, 127), 1.0) == (0.0, 0.0)
    assert pc.expand64_bound(np.r_[0.0, 1.0], 0.0) == (0.0, 0.0)
    assert pc.expand64_bound(np.r_[0.0, 1.0], np.inf) == (0.0, 0.0)


def on_sky(vi, vj, delta):
    """((pi, rp^2) of the form, of the definition, |L|^2); delta: relative error of
    the hardware's reciprocal root before its Newton step."""
    d = [x - y for x, y in zip(vi, vj)]
    ss = fma(d[2], d[2], fma(d[1], d[1], d[0] * d[0]))
    sv = 2.0 * fma(d[2], vi[2], fma(d[1], vi[1], d[0] * vi[0]))
    A4 = 4.0 * ((vi[0] * vi[0] + vi[1] * vi[1]) + vi[2] * vi[2])
    sl = sv - ss
    ll = (A4 - sv) - sl
    r = ll ** -0.5 * (1.0 + delta)
    r = fma(0.5 * r, fma(-(ll * r), r, 1.0), r)
    p = abs(sl) * r
    form = p, max(fma(-p, p, ss), 0.0)
    L = [x + y for x, y in zip(vi, vj)]
    s0 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
    sl = (d[0] * L[0] + d[1] * L[1]) + d[2] * L[2]
    l0 = (L[0] * L[0] + L[1] * L[1]) + L[2] * L[2]
    p = abs(sl) / float(np.sqrt(l0)) if l0 > 0.0 else 0.0
    return form, (p, max(s0 - p * p, 0.0)), ll


@pytest.mark.parametrize("near,far", [(400.0, 1500.0), (20.0, 60.0), (1e5, 1.2e5)])
def test_on_sky_within_its_bounds(near, far):
    edges, pimax, npi = np.logspace(-1.0, np.log10(25.0), 10), 40.0, 40
    ds, dpi = pc.mocks_bounds(edges, pimax, npi, far * far)
    assert ds > 0.0 and dpi > 0.0
    R = np.sqrt(edges[-1] ** 2 + pimax ** 2)
    rng = synth.rng_for(int(far))
    n = 5000
    v = rng.normal(size=(n, 3))
    v *= (rng.uniform(near, far, n) / np.linalg.norm(v, axis=1))[:, None]
    w = rng.normal(size=(n, 3))
    w *= (R * rng.random(n) ** 0.5 / np.linalg.norm(w, axis=1))[:, None]
    w[: n // 4] = v[: n // 4] * (pimax * rng.random(n // 4)
                                 / np.linalg.norm(v[: n // 4], axis=1))[:, None]   # radial
    w[:20] = 0.0
    worst = [0.0, 0.0]
    for k in range(n):
        vi, vj = v[k].tolist(), (v[k] + w[k]).tolist()
        form, exact, ll = on_sky(vi, vj, (1, -1)[k & 1] * 2.0 ** -23)
        if not ll >= far * far / 16.0:
            continue
        worst[0] = max(worst[0], abs(form[0] - exact[0]) / dpi)
        worst[1] = max(worst[1], abs(form[1] - exact[1]) / ds)
    print("on-sky: largest shares of the bounds (pi, rp^2)", worst)
    # the root's error after the step alone, 2^-45.4 of pi, is 2^-8 of dpi
    assert 2.0 ** -9 < worst[0] < 0.125 and 2.0 ** -10 < worst[1] < 0.125


def test_on_sky_limits():
    e = np.array([0.01, 25.0])
    assert pc.mocks_bounds(e, 40.0, 40, 1e6)[0] > 0.0
    # the smallest edge against the reach, pi bins against its error
    assert pc.mocks_bounds(np.array([1e-7, 25.0]), 40.0, 40, 1e6) == (0.0, 0.0)
    assert pc.mocks_bounds(e, 1e6, 40, 1e14) == (0.0, 0.0)
    # observer's distances against the reach, and at the ends of the range
    assert pc.mocks_bounds(e, 40.0, 40, 1e-4) == (0.0, 0.0)
    assert pc.mocks_bounds(e, 40.0, 40, 2.0 ** 201) == (0.0, 0.0)
    assert pc.mocks_bounds(e * 1e-70, 4e-69, 40, 1e-134) == (0.0, 0.0)


@pytest.mark.parametrize("V,spread", [(0.0, 1.0), (1e-3, 1.0), (1.0, 10.0), (30.0, 47.0),
                                      (47.0, 47.0), (1e3, 47.0), (1e5, 47.0)])
def test_on_sky_bounds_by_the_lane(V, spread):
    """The bounds hold for every pair with |L|^2 >= |v_i|^2 / 4 + 2^-60 R^2, however far
    the farthest point of the call lies: lanes at the observer, near it against the
    reach and far from it, pairs on one side of the observer and across it."""
    edges, pimax, npi = np.logspace(-1.0, np.log10(25.0), 10), 40.0, 40
    R2 = edges[-1] ** 2 + pimax ** 2
    ds, dpi = pc.mocks_bounds(edges, pimax, npi, 1e12)
    rng = synth.rng_for(int(V + spread))
    v = rng.normal(size=(3000, 3))
    v *= V / np.linalg.norm(v, axis=1)[:, None]
    w = rng.normal(size=v.shape)
    w *= (spread * 10.0 ** rng.uniform(-3, 0, len(w)) / np.linalg.norm(w, axis=1))[:, None]
    w[::4] = -2.0 * v[::4] * (1.0 - rng.uniform(-0.6, 0.6, len(w[::4])))[:, None]   # across
    worst, used = [0.0, 0.0], 0
    for k in range(len(v)):
        vi, vj = v[k].tolist(), (v[k] + w[k]).tolist()
        if not (w[k] ** 2).sum() < R2 or not np.any(v[k] * 2 + w[k]):
            continue
        form, exact, ll = on_sky(vi, vj, (1, -1)[k & 1] * 2.0 ** -23)
        if not ll >= float((v[k] ** 2).sum()) / 4 + 2.0 ** -60 * R2:
            continue
        used += 1
        worst[0] = max(worst[0], abs(form[0] - exact[0]) / dpi)
        worst[1] = max(worst[1], abs(form[1] - exact[1]) / ds)
    print("on-sky lanes at", V, ": shares of the bounds (pi, rp^2)", worst, used)
    assert used > 500 and worst[0] < 0.125 and worst[1] < 0.125
