"""The x/y refinement chosen by default: dense, large inputs take columns
narrower than the reach, short lists, batches and angular counts do not, and
counts and sums equal those of every explicit refinement."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pc():
    import paper_1911_03545_amd as m
    ctx = m.PairCounter(0)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("stat", ["r", "rppi", "cross", "open"])
def test_chosen_equals_explicit(pc, prec, stat):
    L, e = 80.0, synth.log_edges(0.1, 20.0, 12)
    p = synth.clustered_box(120_000, L, seed=1, nblobs=300)
    q = synth.uniform_box(60_000, L, seed=2)
    w, wq = synth.uniform_weights(len(p), seed=3), synth.uniform_weights(len(q), seed=4)

    def call(k, weighted):
        o = {"xy_refine": k}
        ws = dict(w1=w if weighted else None)
        if stat == "rppi":
            return pc.count_rppi(p, None, e, 20.0, 20, L, prec, options=o, **ws)
        d2 = q if stat == "cross" else None
        if d2 is not None and weighted:
            ws["w2"] = wq
        return pc.count_r(p, d2, e, 0.0 if stat == "open" else L, prec, options=o, **ws)

    for weighted in (False, True):
        got, gw = call(0, weighted)
        chosen = pc.stats()["xy_refine"]
        assert chosen >= 2
        for k in (1, 2, 3):
            want, ww = call(k, weighted)
            assert np.array_equal(got, want), (k, chosen)
            if weighted:
                assert np.all(np.abs(gw - ww) <= 1e-12 * np.abs(ww))


def test_not_refined(pc):
    e = synth.log_edges(0.1, 10.0, 8)
    pc.count_r(synth.uniform_box(3000, 100.0, seed=1), None, e, 100.0, "fp32")
    assert pc.stats()["xy_refine"] == 1
    cats = [synth.uniform_box(n, 60.0, seed=n) for n in (20000, 500)]
    pc.count_rppi_batch(cats, e, 10.0, 10, 60.0, "fp32")
    assert pc.stats()["xy_refine"] == 1
