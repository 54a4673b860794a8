"""count_pairs_r_noalloc near the end of its fixed scratch (needs an MI355X).

790000 host points in binary64 leave about a MiB of the 128 MiB: the call must
take the plan that needs the least scratch and give the counts of the ordinary
entry point.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, prec", [(790_000, "fp64"), (690_000, "fp32")])
def test_largest_catalogues_fit(n, prec):
    import paper_1911_03545_amd as m
    print("noalloc near the limit", n, prec, flush=True)
    e = np.linspace(0.5, 12.0, 8)
    pts = np.random.default_rng(1).random((n, 3)) * 420.0
    ctx = m.PairCounter(0)
    try:
        want, _ = ctx.count_r(pts, None, e, 420.0, prec)
        got, _ = ctx.count_r_noalloc(pts, None, e, 420.0, prec)
    finally:
        ctx.close()
    assert want.sum() > 0
    assert (got == want).all()
