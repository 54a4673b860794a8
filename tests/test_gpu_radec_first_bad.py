"""The first point out of range decides the error of an RA/DEC call, also where
several points of one slab (131072 points) of the host conversion are bad and the
later one is met first by another thread: the first bad point ends a piece (2048
points), the second begins the next one."""
import numpy as np
import pytest

import paper_1911_03545_amd as pc
import synth

pytestmark = pytest.mark.gpu

SLAB, PIECE = 131072, 2048


@pytest.mark.parametrize("slab", [0, 1, 2])
@pytest.mark.parametrize("device", [False, True])
def test_bad_points_in_one_slab(slab, device):
    n = 3 * SLAB
    m = synth.sky_mock(n, seed=5, clustered=False)
    first = slab * SLAB + PIECE - 1
    cols = []
    for ra_at, d_at, want in ((first, first + 1, pc.CF_ERANGE), (first + 1, first, pc.CF_EINVAL)):
        ra, dec, d = (np.array(m[:, k]) for k in range(3))
        ra[ra_at::PIECE] = 361.0       # (and one in every piece after it)
        d[d_at::PIECE] = -1.0
        if device:
            import torch
            ra, dec, d = (torch.from_numpy(a).cuda() for a in (ra, dec, d))
        cols.append(((ra, dec, d), want))
    with pc.PairCounter(0) as ctx:
        for _ in range(60):
            for c, want in cols:
                with pytest.raises(pc.PairCountError) as err:
                    ctx.count_rppi_mocks(c, None, np.array([0.5, 1.0]), 2.0, 2)
                assert err.value.status == want
