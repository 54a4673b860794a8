"""Candidate pairs and blocks that a call reports (needs an MI355X): exact where all
points lie within one reach of each other in an open box of one column, for work
lists in block order and in one pass, first, repeated, and batched calls."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 5000, 65536, 65537, 90001])
def test_single(prec, n):
    import paper_1911_03545_amd as pcm
    p = synth.uniform_box(n, 1.0, seed=n)
    e = np.array([0.001, 0.002, 2.0]) if n < 6000 else np.array([1.9, 2.0])
    with pcm.PairCounter(0) as pc:
        for _ in range(3):
            pc.count_r(p, None, e, 0.0, prec)
            st = pc.stats()
            assert st["candidate_pairs"] == n * (n - 1) // 2
            assert st["n_blocks"] == -(-n // 64)
        q = p[: n // 2 + 1]
        for _ in range(2):
            pc.count_r(p, q, e, 0.0, prec)
            st = pc.stats()
            assert st["candidate_pairs"] == n * len(q)
            assert st["n_blocks"] == -(-n // 64)


def test_batch():
    import paper_1911_03545_amd as pcm
    ns = (1, 64, 700, 65)
    cats = [synth.uniform_box(n, 1.0, seed=n) for n in ns]
    with pcm.PairCounter(0) as pc:
        for _ in range(2):
            pc.count_rppi_batch(cats, np.array([0.5, 2.0]), 2.0, 4, 0.0, "fp32")
            st = pc.stats()
            assert st["candidate_pairs"] == sum(n * (n - 1) // 2 for n in ns)
            assert st["n_blocks"] == sum(-(-n // 64) for n in ns)
