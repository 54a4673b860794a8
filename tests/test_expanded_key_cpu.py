"""Table keys of near pairs in the expanded float32 forms, emulated on the CPU.

The expanded sums round relative to the columns' widths, so the sum of a near
pair can come out below zero: by less than half a cell of the rounding key
where columns are up to twice the reach wide, by many cells where a domain of
thousands of reaches makes them wider (the form is not taken there), and by
whole cells of the linear key (batches, 16-bit tables), which clamps at zero.
Every key is then a cell of the table, and lies on the same side of every edge
as the binary64 separation or in a cell that the edge's band meets; without the
rule and the clamp keys lie past the table (rounding key, read as an unsigned
half) or in the last cell (linear key, clamped by bit pattern)."""
import numpy as np
import pytest

import paper_1911_03545_amd as pc
from test_fp32_contract import U32, expand_mag, fma32


def expanded_sums(box, edges, ndim, linear, n=100_000):
    """Expanded float32 sums of near and coincident pairs of a periodic box,
    their binary64 separations, and the bands, in the sweep's scale."""
    R = edges[-1]
    g = pc.plan_grid_refined(None, None, box, R, R, 32, 1, ndim == 3)
    w = g["width"][0]
    xy_max = [1.5 * w, 1.5 * w, 0.5 * w, 0.5 * w]
    eps = [U32 * 2.0 * w * (1 + 2.0 ** -20) + 2.0 ** -50 * box] * 2 + [
        U32 * (2 * box + R) * (1 + 2.0 ** -20) + 2.0 ** -50 * box]
    lo, hi = pc.fp32_bands_xy(edges ** 2, eps, xy_max, box, ndim)
    top = 16383.0 if linear else 32766.0 / 32767.0
    c = np.sqrt(top * (1.0 - 2.0 ** -16) / float(hi[-1]))
    rng = np.random.default_rng(int(box) + ndim)
    p = rng.uniform(0.0, box, (n, 3))
    q = np.clip(p + rng.normal(size=p.shape) * 1e-3 * R, 0.0, np.nextafter(box, 0.0))
    q[: n // 4] = p[: n // 4]
    centre = (np.floor(q[:, :2] / w) + 0.5) * w
    a, b = (((v[:, :2] - centre) * c).astype(np.float32) for v in (p, q))
    za, zb = ((v[:, 2] * c).astype(np.float32) for v in (p, q))
    A, B = (fma32(v[:, 1], v[:, 1], v[:, 0] * v[:, 0]) for v in (a, b))
    e = np.float32(-2) * a
    if ndim == 3:
        dz = za - zb
        t = fma32(e[:, 1], b[:, 1], fma32(e[:, 0], b[:, 0], fma32(dz, dz, B)))
        s = t + A
    else:
        s = fma32(e[:, 1], b[:, 1], fma32(e[:, 0], b[:, 0], A + B))
    s64 = ((p - q)[:, :ndim] ** 2).sum(1)
    return s, s64, lo.astype(np.float64) * c * c, hi.astype(np.float64) * c * c


def rounding_key(s):
    """round(clamp(s, -1, 1) 32767) as a signed half, read as an unsigned one."""
    return np.rint(np.clip(s, -1.0, 1.0) * np.float32(32767)).astype(np.int16).view(np.uint16)


def linear_key(s, kmax=16383.0):
    return np.clip(s, np.float32(0), np.float32(kmax)).astype(np.int64)


def by_bits(s, kmax=16383.0):
    return np.minimum(s.view(np.uint32), np.float32(kmax).view(np.uint32)).view(
        np.float32).astype(np.int64)


# (domains of 1024 columns 2.42 and 2.11 reaches wide: where kSafety u times the
# magnitude term, 17.5 and 23 squared widths, meets 2^-17 of the squared reach)
WIDEST = {n: 1024 * np.sqrt(2.0 ** -17 / (1.25 * U32 * m)) for n, m in ((3, 17.5), (2, 23.0))}
CASES = [(WIDEST[3], 0.02, 3, False), (WIDEST[2], 0.06, 2, False), (100.0, 0.1, 3, False),
         (100.0, 0.1, 2, False), (100.0, 0.1, 2, True), (100.0, 0.1, 3, True),
         (3.0e4, 0.02, 3, True), (1.0e5, 0.4, 2, True)]


@pytest.mark.parametrize("box,first,ndim,linear", CASES)
def test_keys_inside_the_table(box, first, ndim, linear):
    reach = 10.0 if box == 100.0 else 1.0
    edges = np.r_[0.0, np.logspace(np.log10(first), np.log10(reach), 11)]
    s, s64, lo, hi = expanded_sums(box, edges, ndim, linear)
    assert (s < 0).any()
    if linear:
        key, width, last = linear_key(s), 1.0, 16383
        cell_lo, cell_hi = key, key + 1.0
    else:
        key, width, last = rounding_key(s).astype(np.int64), 1 / 32767, 32767
        cell_lo, cell_hi = (key - 0.5) * width, (key + 0.5) * width
    assert key.min() >= 0 and key.max() <= last
    for k in range(1, len(edges)):     # (the band of the zero edge is empty)
        below, above = cell_hi < lo[k], cell_lo > hi[k]
        assert not (below & (s64 >= edges[k] ** 2)).any()
        assert not (above & (s64 < edges[k] ** 2)).any()


def test_keys_outside_the_rules():
    """What the rule and the clamp are for: a near pair of the first bin keyed past
    the table, or into its last cell, which lies above every edge."""
    s, _, _, _ = expanded_sums(3.0e4, np.r_[0.0, np.logspace(np.log10(0.02), 0, 11)], 3, False)
    assert (rounding_key(s) > 32767).sum() > 100
    s, _, _, _ = expanded_sums(100.0, np.r_[0.0, np.logspace(-1, 1, 11)], 2, True)
    assert (by_bits(s) == 16383).sum() > 100
