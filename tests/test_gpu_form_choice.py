"""The default separation form of float32 DD(r) against the oracle (needs an
MI355X): expanded up to a rounding term of 4 times the smallest nonzero squared
edge, differences beyond it and, past an eighth, for tables of 16 bits.  Columns
here are 10 wide, so the term is 1.7e-4 (k = 1).
"""
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


@pytest.mark.parametrize("box", [100.0, 0.0])
@pytest.mark.parametrize("lo, nb, zero, form", [
    (0.05, 20, False, 2),    # 0.07 times the first edge squared
    (0.02, 20, False, 2),    # 0.4
    (0.008, 20, False, 2),   # 2.6
    (0.008, 20, True, 2),    # a zero edge below it
    (0.004, 20, False, 1),   # 10
    (0.008, 125, False, 2),  # the most bins of a byte table
    (0.02, 126, False, 1),   # 16-bit table
])
def test_default_form(pc, box, lo, nb, zero, form):
    print("default form", box, lo, nb, zero, flush=True)
    x = synth.clustered_box(20000, 100.0, seed=1401, nblobs=200, sigma=0.3)
    x[:100] = x[100:200]                      # coincident pairs
    x[200:300] = np.clip(x[300:400] + 1e-6, 0.0, 99.999)   # and nearly so
    w = synth.uniform_weights(20000, 1402)
    e = synth.log_edges(lo, 9.99, nb - zero)
    e = np.r_[0.0, e] if zero else e
    opt = {"xy_refine": 1}
    want, ww = oracle.count_r(x, None, e, box, w1=w)
    got, gw = pc.count_r(x, None, e, box, "fp32", w1=w, options=opt)
    assert pc.stats()["separation_form"] == form
    assert (got == want).all()
    # binary64 sums of at most 4e8 products by atomics
    np.testing.assert_allclose(gw, ww, rtol=1e-12, atol=0)
    got, _ = pc.count_r(x, None, e, box, "fp32", options=opt)
    assert (got == want).all()
    y = x[:5000] + 0.0
    want, _ = oracle.count_r(x, y, e, box)
    got, _ = pc.count_r(x, y, e, box, "fp32", options=opt)
    assert (got == want).all()
