"""Radiation moments at the edges of their tiles (64 x 16 cells in 2D, 64 x 4 x 4 in 3D, a thread's
four cells a column of planes): one cell below, at and above them, and columns cut by the level's
top, against the oracle at the bounds of test_gpu_moments."""
import pytest

import workloads as W
from tests.test_gpu_moments import check, run

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (4, 4, 64), (5, 3, 65), (3, 5, 63), (9, 6, 66), (2, 64), (16, 64), (17, 65), (15, 63), (33, 3)]


@pytest.mark.parametrize("limiter", ["lp", "minerbo"])
def test_moments_at_tile_edges_match_the_oracle(limiter):
    grids = [W.random_grid(s, 91000 + i, dt=1e-3) for i, s in enumerate(SHAPES)]
    res = run(grids, limiter=limiter)
    for i, g in enumerate(grids):
        check.index = i
        check(g, res[i], 1.0, limiter, True)
