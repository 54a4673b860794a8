"""Device scratch of binary64 cross-correlations (needs an MI355X): the expanded form
keeps |b|^2 for the second side alone and neither side's float32 coordinates, so
it takes no more than the differences."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def taken(shift, n1, n2):
    """Bytes a fresh context asks for, and the form it takes."""
    import torch
    import paper_1911_03545_amd as pcm
    live, total = {}, [0]

    def alloc(n):
        t = torch.empty(n + 256, dtype=torch.uint8, device="cuda:0")
        p = (t.data_ptr() + 255) // 256 * 256
        live[p] = t
        total[0] += n
        return p

    p, q = (synth.uniform_box(n, 40.0, seed=n) + shift for n in (n1, n2))
    e = np.array([0.1, 1.0, 2.0])
    with pcm.PairCounter(0) as pc:
        pc.set_allocator(alloc, lambda a: live.pop(a, None))
        got, _ = pc.count_r(p, q, e, 0.0, "fp64")
        form = pc.binary64_form()
    want, _ = oracle.count_r_pruned(p, q, e, 0.0)
    assert np.array_equal(got, want)
    return total[0], form


@pytest.mark.parametrize("n1,n2", [(200_000, 1000), (1000, 200_000)])
def test_scratch(n1, n2):
    expanded, f2 = taken(0.0, n1, n2)
    differences, f1 = taken(1.0e6, n1, n2)
    assert (f2, f1) == (2, 1)
    # three float32 columns of either side less, 8 bytes per second point more
    # (buffers hold a quarter of headroom; the rest is of the same size within 1%)
    assert expanded <= differences + 10 * n2 - 15 * (n1 + n2) + differences // 100
