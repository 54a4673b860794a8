"""The default x/y refinement (cf_plan_refine) prices the grids that are built: no
columns narrower than 1024 an axis allow, slices as far apart as 2^26 cells allow."""
import math

import numpy as np
import pytest

import paper_1911_03545_amd as pc


def cost(ext, reach, n, k, item=2500.0):
    """Pairs and items a block of 64 points costs on the grid built for k (an open
    box of evenly spread points, the reach a ball)."""
    g = pc.plan_grid_refined([0.0] * 3, ext, 0.0, reach, reach, 32, k, True)
    (wx, wy, wz), rho = g["width"], n / np.prod(ext)
    b = min(64.0 / (rho * wx * wy), ext[2])
    # a window ends on slices: besides those asked for, what coarser ones add
    coarse = 2.0 * (wz - reach / 32) if wz > 1.5 * reach / 32 else 0.0
    c = 6000.0 * (k - 1)
    for ox in range(-k, k + 1):
        for oy in range(-k, k + 1):
            d2 = (max(abs(ox) - 1, 0) * wx) ** 2 + (max(abs(oy) - 1, 0) * wy) ** 2
            if d2 < reach * reach:
                z = 2.0 * math.sqrt(reach * reach - d2) + b + coarse
                c += 64 * rho * wx * wy * min(z, ext[2]) + item
    return c


@pytest.mark.parametrize("ext", [[100.0] * 3, [150.0] * 3, [300.0] * 3, [3000.0, 10.0, 10.0],
                                 [2000.0, 5.0, 5.0], [5000.0, 5.0, 500.0], [600.0, 600.0, 3.0],
                                 [3000.0, 3000.0, 4.0]])
@pytest.mark.parametrize("n", [1e7, 1e8, 1e9, 2e9])
def test_built_grids_are_priced(ext, n):
    k = pc.plan_refine([0.0] * 3, ext, 0.0, 1.0, 1.0, n)
    costs = {q: cost(ext, 1.0, n, q) for q in (1, 2, 3, 4)}
    # (a refinement is taken for 3% of the least before it)
    assert costs[k] <= min(costs.values()) / 0.97, costs


@pytest.mark.parametrize("ext,n,k", [
    ([150.0] * 3, 1e9, 1),           # finer columns would coarsen the slices
    ([600.0, 600.0, 3.0], 2e9, 2),   # 1024 columns an axis: 3 is 2 again
    ([2000.0, 5.0, 5.0], 1e7, 2),    # columns of two reaches along x at any k
])
def test_where_the_caps_decide(ext, n, k):
    assert pc.plan_refine([0.0] * 3, ext, 0.0, 1.0, 1.0, n) == k


def test_ordinary_boxes():
    for reach, ball, item, k in ((25.0, True, 2500.0, 1), (25.0, True, 1250.0, 2),
                                 (50.0, True, 4300.0, 3)):
        assert pc.plan_refine(None, None, 420.0, reach, reach, 1e6, None, item, 32, ball) == k
    assert pc.plan_refine(None, None, 420.0, 25.0, 40.0, 1e6, None, 2000.0, 32, False) == 2
    assert pc.plan_refine(None, None, 100.0, 10.0, 10.0, 1e4) == 1
    with pytest.raises(pc.PairCountError):
        pc.plan_refine(None, None, 0.0, 10.0, 10.0, 1e4)
