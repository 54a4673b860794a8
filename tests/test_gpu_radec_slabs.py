"""RA/DEC converted on the host in slabs of pinned memory: the vectors of
every point, at sizes around a piece (2048) and a slab (131072) of the
conversion and beyond the slabs kept in flight, from device and host columns
of both types.  Counts from RA/DEC equal the counts from the oracle's unit
vectors bit for bit (the same C library functions), and the first point out of
range decides the error."""
import numpy as np
import pytest

import oracle
import paper_1911_03545_amd as pc
import synth

pytestmark = pytest.mark.gpu

EDGES = np.array([0.02, 0.05, 0.11])


def columns(cols, dtype, device):
    cols = [np.ascontiguousarray(c, dtype=dtype) for c in cols]
    if not device:
        return cols
    import torch
    return [torch.from_numpy(c).cuda() for c in cols]


@pytest.mark.parametrize("n", [1, 2047, 2049, 131071, 131073, 3 * 131072 + 5, 600001])
@pytest.mark.parametrize("dtype,device", [(np.float64, True), (np.float32, True),
                                          (np.float64, False), (np.float32, False)])
def test_slabs_equal_unit_vectors(n, dtype, device):
    ra, dec = synth.cap_radec(n, seed=n % 97, radius_deg=20.0, clustered=n > 10, nblobs=50)
    ra, dec = (np.asarray(a, dtype=dtype) for a in (ra, dec))
    ra = np.minimum(ra, dtype(360.0))
    v = oracle.radec_to_unit(ra.astype(np.float64), dec.astype(np.float64))
    with pc.PairCounter(0) as ctx:
        want, _ = ctx.count_theta(None, None, None, None, EDGES, "fp64",
                                  unit_vectors=(np.ascontiguousarray(v), None))
        for _ in range(2):   # the second call reuses the slabs
            got, _ = ctx.count_theta(*columns((ra, dec), dtype, device), None, None, EDGES,
                                     "fp64")
            assert np.array_equal(got, want)


@pytest.mark.parametrize("device", [True, False])
def test_first_bad_point_decides(device):
    n = 300000
    m = synth.sky_mock(n, seed=3, clustered=False)
    e = np.array([0.5, 1.0])
    with pc.PairCounter(0) as ctx:
        for at_ra, at_d, want in ((290000, 1000, pc.CF_EINVAL), (1000, 290000, pc.CF_ERANGE),
                                  (299999, None, pc.CF_ERANGE), (None, 299999, pc.CF_EINVAL)):
            ra, dec, d = (np.array(m[:, k]) for k in range(3))
            if at_ra is not None:
                ra[at_ra] = 361.0
            if at_d is not None:
                d[at_d] = np.nan
            with pytest.raises(pc.PairCountError) as err:
                ctx.count_rppi_mocks(tuple(columns((ra, dec, d), np.float64, device)), None, e,
                                     2.0, 2)
            assert err.value.status == want
        # and the context works afterwards
        cols = tuple(columns([m[:, k] for k in range(3)], np.float64, device))
        a, _ = ctx.count_rppi_mocks(cols, None, e, 2.0, 2)
        v = oracle.sky_to_cartesian(m[:, 0], m[:, 1], m[:, 2])
        b, _ = ctx.count_rppi_mocks(np.ascontiguousarray(v), None, e, 2.0, 2, cartesian=True)
        assert np.array_equal(a, b)
