"""The default x/y refinement of binary64 DD(r) is the same with and without weights
(needs an MI355X): at 10^6 points of reach 25 in a box of 420 columns of half a reach
pay either way, at half the density they do not."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,want", [(1_000_000, 2), (500_000, 1)])
def test_same_with_weights(n, want):
    import torch
    import paper_1911_03545_amd as pcm
    L, e = 420.0, synth.log_edges(0.1, 25.0, 20)
    p = synth.clustered_box(n, L, seed=1, nblobs=n // 200)
    cols = [torch.from_numpy(np.ascontiguousarray(p[:, k])).cuda() for k in range(3)]
    w = torch.from_numpy(synth.uniform_weights(n, seed=3)).cuda()
    with pcm.PairCounter(0) as pc:
        plain, _ = pc.count_r(cols, None, e, L, "fp64")
        assert pc.stats()["xy_refine"] == want
        for kw in (dict(w1=w), dict(w1=w, options={"deterministic_weights": 1}),
                   dict(ravg=True)):
            got = pc.count_r(cols, None, e, L, "fp64", **kw)[0]
            assert pc.stats()["xy_refine"] == want and np.array_equal(got, plain)
