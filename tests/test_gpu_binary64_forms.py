"""Which form the binary64 sweeps take, and that pairs within its error bound of an
edge are decided by the definition and counted (needs an MI355X): the expanded
DD(r) from the origin out to where its bound outgrows the smallest edge, the
on-sky form and the inputs that return to the definition, graph replays, float32
and empty calls."""
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


@pytest.mark.parametrize("shift,form", [(0.0, 2), (1e3, 2), (2e4, 2), (3e4, 1), (1e9, 1)])
def test_expanded_r(pc, shift, form):
    p = synth.lattice_box(3000, 16, seed=4, denom=4) + shift   # ties with the edges
    e = np.array([0.25, 0.75, 1.25, 3.0])
    want, _ = oracle.count_r(p, None, e, 0.0)
    got, _ = pc.count_r(p, None, e, 0.0, "fp64")
    assert np.array_equal(got, want)
    assert pc.binary64_form() == form
    assert (pc.stats()["rechecks"] > 0) == (form == 2)
    assert pc.stats()["separation_form"] == 0
    for kw in (dict(w1=np.ones(len(p))), dict(ravg=True)):   # the differences
        assert np.array_equal(pc.count_r(p, None, e, 0.0, "fp64", **kw)[0], want)
        assert pc.binary64_form() == 1
    assert np.array_equal(pc.count_r(p, None, e, 0.0, "fp32")[0], want)
    assert pc.binary64_form() == 0


def test_expanded_chords(pc):
    ra, dec = synth.cap_radec(3000, seed=2, radius_deg=20.0)
    e = np.array([0.05, 1.0, 5.0])
    for ang in (0, -1):
        got, _ = pc.count_theta(ra, dec, None, None, e, "fp64", angular_grid=ang)
        assert np.array_equal(got, oracle.count_theta(ra, dec, None, None, e)[0])
        assert pc.binary64_form() == 2
    # 2^-12 of the smallest squared chord is below the bound
    pc.count_theta(ra, dec, None, None, np.array([1e-5, 5.0]), "fp64")
    assert pc.binary64_form() == 1


@pytest.mark.parametrize("first,npi,form", [(0.25, 8, 2), (1e-8, 8, 1)])
def test_on_sky(pc, first, npi, form):
    rng = synth.rng_for(6)
    p = rng.integers(0, 13, size=(1500, 3)).astype(np.float64)
    p[::3, :2] = 0.0
    p[:, 2] += 40.0
    e = np.array([first, 1.0, 4.0])
    want, _ = oracle.count_rppi_mocks(p, None, e, 8.0, npi)
    for prec in ("fp64", "fp32"):   # (on-sky pairs are binary64 in both modes)
        got, _ = pc.count_rppi_mocks(p, None, e, 8.0, npi, prec, cartesian=True)
        assert np.array_equal(got, want)
        assert pc.binary64_form() == form
        assert (pc.stats()["rechecks"] > 0) == (form == 2)
    got = pc.count_rppi_mocks(p, None, e, 8.0, npi, "fp64", cartesian=True, ravg=True)[0]
    assert np.array_equal(got, want) and pc.binary64_form() == 1


def test_replayed_and_empty(pc):
    import torch
    p = synth.lattice_box(3000, 16, seed=9, denom=4)
    cols = [torch.from_numpy(np.ascontiguousarray(p[:, k])).cuda() for k in range(3)]
    e = np.array([0.25, 0.75, 3.0])
    for _ in range(3):
        pc.count_r(cols, None, e, 16.0, "fp64", options={"use_graph": 1})
        assert pc.binary64_form() == 2 and pc.stats()["rechecks"] > 0
    assert pc.stats()["replayed"] == 1
    pc.count_r(np.zeros((0, 3)), None, e, 16.0, "fp64")
    assert pc.binary64_form() == 0
