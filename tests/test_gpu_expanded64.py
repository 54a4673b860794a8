"""The binary64 r sweep with the squared separation expanded (|a|^2 + |b|^2 -
2 a.b): counts equal to the definition's, on lattices with exact edge ties,
with coincident points under a first edge of zero, at sizes around a block (64)
and a chunk (8), for auto- and cross-correlations, periodic and shifted far
from the origin (where the form's error outgrows the edges and the sweep
returns to differences), with one replica per lane and with shared ones."""
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


def lattice(n, seed):
    """Points on quarters with some coincident ones: separations tie edges."""
    p = synth.lattice_box(n, 16, seed, denom=4)
    p[n // 2:n // 2 + n // 8] = p[:n // 8]
    return p


EDGES = [np.array([0.0, 0.25, 0.5, 1.0, 1.5, 2.5, 4.0]), np.array([0.25, 0.75, 1.25, 3.0]),
         np.array([0.0, 4.5])]


@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 129, 1500])
@pytest.mark.parametrize("k", range(len(EDGES)))
@pytest.mark.parametrize("box", [16.0, 0.0])
def test_lattice_ties(pc, olib, n, k, box):
    e = EDGES[k]
    p, q = lattice(n, 11 * n + k), lattice(max(1, n // 2 + 3), 13 * n + k)
    for d2 in (None, q):
        want, _ = oracle.count_r(p, d2, e, box, lib=olib)
        for opts in (None, {"hist_copies": 4}, {"chunk": 64}):
            got, _ = pc.count_r(p, d2, e, box, "fp64", options=opts)
            assert np.array_equal(got, want), (opts, d2 is None)


@pytest.mark.parametrize("shift", [0.0, 1.0e3, 1.0e5, 1.0e7, 1.0e9])
def test_shifted_from_the_origin(pc, olib, shift):
    rng = synth.rng_for(77)
    p = rng.uniform(0.0, 12.0, size=(3000, 3))
    p[:40] = p[40:80] + 1.0e-9   # below the first edge, or just past it
    p += shift
    e = np.r_[0.0, np.logspace(-3, np.log10(3.0), 17)]
    want, _ = oracle.count_r(p, None, e, 0.0, lib=olib)
    got, _ = pc.count_r(p, None, e, 0.0, "fp64")
    assert np.array_equal(got, want)


@pytest.mark.parametrize("scale", [1.0e-6, 1.0, 1.0e6])
def test_scaled(pc, olib, scale):
    p = synth.clustered_box(4000, 20.0, seed=5, nblobs=30, sigma=0.5) * scale
    p = np.minimum(p, 20.0 * scale)
    e = synth.log_edges(0.02, 5.0, 125) * scale
    want, _ = oracle.count_r(p, None, e, 20.0 * scale, lib=olib)
    got, _ = pc.count_r(p, None, e, 20.0 * scale, "fp64")
    assert np.array_equal(got, want)
