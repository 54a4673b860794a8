"""On-sky counts of catalogues whose farthest point lies far beyond the others, and of
points mostly near the observer (needs an MI355X): the counts of the definition, and
pairs decided by it no more common than without the outlier."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["outlier", "near"])
@pytest.mark.parametrize("weighted", [False, True])
def test_few_pairs_by_the_definition(kind, weighted):
    import paper_1911_03545_amd as pcm
    m = synth.sky_mock(6000, seed=8)
    p = oracle.sky_to_cartesian(m[:, 0], m[:, 1], m[:, 2])
    rng = synth.rng_for(9)
    if kind == "outlier":
        p = np.vstack([p, [[3.0e4, 0.0, 0.0]]])
    else:
        p = p * rng.uniform(0.02, 1.0, len(p))[:, None] ** 2
    w = dict(w1=synth.uniform_weights(len(p), 10)) if weighted else {}
    e = synth.log_edges(0.1, 25.0, 14)
    want, ww = oracle.count_rppi_mocks(p, None, e, 40.0, 40, **w)
    with pcm.PairCounter(0) as pc:
        got, gw = pc.count_rppi_mocks(p, None, e, 40.0, 40, "fp64", cartesian=True, **w)
        assert np.array_equal(got, want)
        if weighted:
            assert np.all(np.abs(gw - ww) <= 1e-12 * np.abs(ww))
        assert pc.binary64_form() == 2
        # pairs across the observer, |L| below half of either distance, and half a
        # percent for pairs near edges; by the farthest point's distance it was
        # nearly every pair
        V2 = (p ** 2).sum(1)
        wide = 0
        for i in range(len(p) - 1):
            s2, L2 = (((p[i + 1:] + f * p[i]) ** 2).sum(1) for f in (-1.0, 1.0))
            wide += int(((s2 <= 25.0 ** 2 + 40.0 ** 2) &
                         (L2 <= np.maximum(V2[i + 1:], V2[i]) / 4 + 1e-9)).sum())
        print(kind, weighted, pc.stats()["rechecks"], wide, "of", int(want.sum()) // 2)
        assert pc.stats()["rechecks"] <= wide + int(want.sum()) // 400
