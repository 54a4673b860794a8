"""Near and coincident pairs in the expanded float32 forms (needs an MI355X):
counts equal to the oracle's where the expanded sum of such a pair rounds below
zero -- domains of thousands of reaches, whose columns (1024 an axis) are many
reaches wide (byte tables return to the differences there), and the linear keys
of batches and 16-bit tables on ordinary domains -- with and without a first
edge at zero, weights, a box, for auto- and cross-correlations."""
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


def groups(n, box, spread, seed):
    """Groups of eight points within about `spread`, two of them coincident."""
    rng = synth.rng_for(seed)
    p = np.repeat(rng.uniform(0.0, box, (n // 8, 3)), 8, axis=0)
    p += rng.normal(size=p.shape) * spread * 10.0 ** rng.uniform(-4.0, 0.0, (len(p), 1))
    p[1::8] = p[::8]
    p[3::8, :2] = p[2::8, :2]      # coincident on the sky plane only
    return np.clip(p, 0.0, np.nextafter(box, 0.0))


def edges(first, reach, nb, zero):
    e = np.logspace(np.log10(first), np.log10(reach), nb + 1)
    return np.r_[0.0, e] if zero else e


@pytest.mark.parametrize("size,first,form", [(3.0e4, 0.02, 0), (1.0e5, 0.06, 0),
                                             (1.0e5, 0.4, 2)])
@pytest.mark.parametrize("zero", [True, False])
@pytest.mark.parametrize("nb", [12, 140])
@pytest.mark.parametrize("periodic", [True, False])
def test_r_wide_domain(pc, olib, size, first, form, zero, nb, periodic):
    print("r wide", size, first, form, zero, nb, periodic, flush=True)
    p, q = groups(4000, size, 0.5, 31), groups(4000, size, 0.5, 31)[::3] + 0.0
    w = synth.uniform_weights(len(p), 32)
    e = edges(first, 1.0, nb, zero)
    box = size if periodic else 0.0
    opt = {"separation_form": form}
    want, ww = oracle.count_r(p, None, e, box, w1=w, lib=olib)
    got, _ = pc.count_r(p, None, e, box, "fp32", options=opt)
    assert np.array_equal(got, want)
    # (by default the 16-bit tables keep the differences here too)
    assert pc.stats()["separation_form"] == (2 if nb > 125 and form == 2 else 1)
    got, gw = pc.count_r(p, None, e, box, "fp32", w1=w, options=opt)
    assert np.array_equal(got, want)
    # binary64 sums of at most 4e4 products, added in any order
    np.testing.assert_allclose(gw, ww, rtol=1e-11, atol=0)
    want, _ = oracle.count_r(p, q, e, box, lib=olib)
    got, _ = pc.count_r(p, q, e, box, "fp32", options=opt)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("size", [100.0, 3.0e4, 1.0e5])
@pytest.mark.parametrize("zero", [True, False])
@pytest.mark.parametrize("nb", [8, 130])
def test_rppi(pc, olib, size, zero, nb):
    print("rppi", size, zero, nb, flush=True)
    reach = 10.0 if size == 100.0 else 1.0
    p = groups(4000, size, 0.3 * reach, 33)
    w = synth.uniform_weights(len(p), 34)
    e = edges(0.2 * reach, reach, nb, zero)
    opt = {"separation_form": 2}
    want, ww = oracle.count_rppi(p, None, e, 2.0, 4, size, w1=w, lib=olib)
    got, gw = pc.count_rppi(p, None, e, 2.0, 4, size, "fp32", w1=w, options=opt)
    assert pc.stats()["separation_form"] == (2 if size == 100.0 or nb > 125 else 1)
    assert np.array_equal(got, want)
    np.testing.assert_allclose(gw, ww, rtol=1e-11, atol=0)
    got, _ = pc.count_rppi(p, None, e, 2.0, 4, size, "fp32", options=opt)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("size", [100.0, 3.0e4])
@pytest.mark.parametrize("form", [0, 2])
@pytest.mark.parametrize("nb", [8, 130])
def test_batch(pc, olib, size, form, nb):
    print("batch", size, form, nb, flush=True)
    reach = 10.0 if size == 100.0 else 1.0
    cats = [groups(n, size, 0.3 * reach, n) for n in (4000, 96, 1600)]
    ws = [synth.uniform_weights(len(p), 35) for p in cats]
    e = edges(0.2 * reach, reach, nb, True)
    opt = {"separation_form": form}
    got, _ = pc.count_rppi_batch(cats, e, 2.0, 4, size, "fp32", options=opt)
    gotw, gw = pc.count_rppi_batch(cats, e, 2.0, 4, size, "fp32", weights=ws, options=opt)
    for k, p in enumerate(cats):
        want, ww = oracle.count_rppi(p, None, e, 2.0, 4, size, w1=ws[k], lib=olib)
        assert np.array_equal(got[k], want) and np.array_equal(gotw[k], want)
        np.testing.assert_allclose(gw[k], ww, rtol=1e-11, atol=0)
