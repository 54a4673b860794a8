"""The sweep's launch of a repeated call (needs an MI355X): the list of the call
before sizes it, but a call of few items does not leave the next one, of the same
shape with a thousand, on a workgroup or two; the counts are those of a first
call."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_few_items_then_many(graph, prec):
    import torch
    import paper_1911_03545_amd as pcm
    n, L, e = 1000, 100.0, np.array([0.5, 2.0, 10.0])
    few = np.full((n, 3), 50.0) + synth.uniform_box(n, 0.4, seed=1)   # one cell
    many = synth.uniform_box(n, L, seed=2)
    cols = [torch.from_numpy(np.ascontiguousarray(few[:, k])).cuda() for k in range(3)]
    opt = {"use_graph": graph, "chunk": 100000}
    with pcm.PairCounter(0) as pc:
        want, _ = pc.count_r(many, None, e, L, prec, options={"chunk": 100000})
        first = pc.stats()
        assert 300 < first["n_items"] < 1000   # (within the room of any repeat)
    with pcm.PairCounter(0) as pc:
        for _ in range(2):
            pc.count_r(cols, None, e, L, prec, options=opt)
        assert pc.stats()["n_items"] < 60
        for k in range(3):
            cols[k].copy_(torch.from_numpy(np.ascontiguousarray(many[:, k])))
        torch.cuda.synchronize()
        got, _ = pc.count_r(cols, None, e, L, prec, options=opt)
        assert np.array_equal(got, want)
        if not graph:   # (a replay reports the launch of the recorded call)
            assert pc.stats()["sweep_workgroups"] >= first["sweep_workgroups"]
