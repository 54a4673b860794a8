"""The j points per work item that a caller asks for (cf_options.chunk) are the
length its items have, on work lists of any size (needs an MI355X).  All points lie
within one reach of each other in an open box of one column, so block b (64 points)
meets the n - 1 - 64 b points after its own first in one run, cut into pieces of
`chunk`."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 1000, 4000])
@pytest.mark.parametrize("chunk", [1, 10, 30, 64, 100, 300, 2047, 100000])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_asked_length(n, chunk, prec):
    import paper_1911_03545_amd as pcm
    p = synth.uniform_box(n, 1.0, seed=n)
    e = np.array([0.0, 0.1, 2.0])
    want, _ = oracle.count_r(p, None, e, 0.0)
    with pcm.PairCounter(0) as pc:
        got, _ = pc.count_r(p, None, e, 0.0, prec, options={"chunk": chunk})
        st = pc.stats()
        assert np.array_equal(got, want)
        runs = n - 1 - np.arange(0, n, 64)
        assert st["chunk"] == chunk
        assert st["n_items"] == sum(-(-r // chunk) for r in runs if r > 0)
        # the default shortens the items of so short a list
        pc.count_r(p, None, e, 0.0, prec)
        assert pc.stats()["n_items"] >= sum(-(-r // 128) for r in runs if r > 0)
