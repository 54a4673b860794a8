"""The autotuner starts from the x/y refinement that an untuned call takes (needs
an MI355X): a dense call tunes to that refinement or a neighbour, a batch to the
plain columns or 2, and an asked refinement is left alone."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def pc():
    import paper_1911_03545_amd as m
    ctx = m.PairCounter(0)
    yield ctx
    ctx.close()


def refinement(pc, opt, p, e, L):
    got, _ = pc.count_r(p, None, e, L, "fp32", options=opt)
    return pc.stats()["xy_refine"], got


def test_dense_call(pc):
    L, e = 100.0, synth.log_edges(0.3, 30.0, 10)
    p = synth.clustered_box(400_000, L, seed=8, nblobs=500)
    chosen, want = refinement(pc, {}, p, e, L)
    assert chosen >= 4
    for _ in range(2):   # the second call takes the stored choice
        tuned, got = refinement(pc, {"autotune": 1}, p, e, L)
        assert abs(tuned - chosen) <= 1 and np.array_equal(got, want)
    tuned, got = refinement(pc, {"autotune": 1, "xy_refine": 2}, p, e, L)
    assert tuned == 2 and np.array_equal(got, want)


def test_batch(pc):
    cats = [synth.uniform_box(n, 60.0, seed=n) for n in (20000, 500)]
    e = synth.log_edges(0.1, 10.0, 8)
    want, _ = pc.count_rppi_batch(cats, e, 10.0, 10, 60.0, "fp32")
    got, _ = pc.count_rppi_batch(cats, e, 10.0, 10, 60.0, "fp32", options={"autotune": 1})
    assert pc.stats()["xy_refine"] in (1, 2) and np.array_equal(got, want)
