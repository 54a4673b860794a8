"""On-sky pairs formed from 2 s.v_i with a one-step reciprocal root: counts
equal to the definition's where that form has to give way -- points near the
observer, on opposite sides of it and at it (|L|^2 small or zero), coincident
and radial pairs, pi edges met exactly, very many and very few pi bins, 16-bit
tables, edges starting at zero, sizes around a block and a chunk -- and weight
sums to the usual tolerance."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pc():
    import paper_1911_03545_amd as m
    ctx = m.PairCounter(0)
    yield ctx
    ctx.close()


@pytest.fixture(scope="module")
def olib():
    return oracle.load()


def points(kind, n, seed):
    rng = synth.rng_for(seed)
    if kind == "round the observer":
        p = rng.normal(0.0, 6.0, size=(n, 3))
        p[: n // 6] *= 1e-3
        p[0] = 0.0
        p[n // 6: n // 3] = -p[n // 3: n // 3 + (n // 3 - n // 6)] * (1.0 + 1e-9)
    elif kind == "far":
        p = np.array([900.0, -700.0, 400.0]) + rng.normal(0.0, 5.0, size=(n, 3))
    elif kind == "near and far":
        d = np.where(rng.uniform(size=n) < 0.5, rng.uniform(0.0, 8.0, n),
                     rng.uniform(50.0, 64.0, n))
        u = rng.normal(size=(n, 3)) * [0.1, 0.1, 0.1] + [0.0, 0.0, 1.0]
        p = u / np.linalg.norm(u, axis=1)[:, None] * d[:, None]
    else:   # integers on an axis and beside it: radial pairs on pi edges
        p = rng.integers(0, 13, size=(n, 3)).astype(np.float64)
        p[::3, :2] = 0.0
        p[:, 2] += 40.0
    if n > 8:
        p[n // 2: n // 2 + n // 8] = p[: n // 8]   # coincident pairs
    return np.ascontiguousarray(p)


@pytest.mark.parametrize("kind", ["round the observer", "far", "near and far", "lattice"])
@pytest.mark.parametrize("n", [1, 9, 64, 65, 1200])
@pytest.mark.parametrize("edges,pimax,npi", [
    (np.array([0.0, 0.5, 1.0, 2.0, 4.0]), 6.0, 6),
    (np.array([0.3, 1.0, 5.0]), 8.0, 1),
    (np.array([0.5, 3.0]), 5.0, 1000),
    (np.r_[0.0, np.logspace(-1.0, 0.7, 130)], 4.0, 2)])
def test_equal_to_the_definition(pc, olib, kind, n, edges, pimax, npi):
    p = points(kind, n, seed=n + npi)
    q = points(kind, max(1, n // 2), seed=n + npi + 1)
    for d2 in (None, q):
        want, _ = oracle.count_rppi_mocks(p, d2, edges, pimax, npi, lib=olib)
        got, _ = pc.count_rppi_mocks(p, d2, edges, pimax, npi, "fp64", cartesian=True)
        assert np.array_equal(got, want), d2 is None
    w = synth.uniform_weights(n, seed=3)
    want, ww = oracle.count_rppi_mocks(p, None, edges, pimax, npi, w1=w, lib=olib)
    got, gw = pc.count_rppi_mocks(p, None, edges, pimax, npi, "fp64", w1=w, cartesian=True)
    assert np.array_equal(got, want)
    assert np.all(np.abs(gw - ww) <= 1e-12 * np.abs(ww))
