"""The start of a step under CG (faces, right-hand side, residual and norms from D in one pass)
against the separate passes that the other solvers keep, at the edges of its tiles: with a
target that the start already meets, the norms and the true residual of what it stored are the
same bits; iterated, the solutions agree as far as the two solvers' targets."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2, run_step

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (4, 4, 64), (5, 3, 65), (3, 5, 63), (9, 6, 66), (2, 2), (2, 64), (16, 64), (17, 65), (15, 63), (33, 3)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("limiter", ["lp", "lp_exact"])
def test_start_matches_the_separate_passes(limiter, precision):
    grids = [W.random_grid(s, 92000 + i, dt=1e-3) for i, s in enumerate(SHAPES)]
    kw = dict(limiter=limiter, precision=precision)
    short = [W.random_grid(s, 92000 + i, dt=1e-9) for i, s in enumerate(SHAPES)]
    xs, a, _ = run_step(short, rtol=0.5, krylov=1, fmg=0, **kw)
    _, b, _ = run_step(short, rtol=0.5, krylov=0, fmg=0, **kw)
    for g, x, s, t in zip(short, xs, a, b):
        assert np.array_equal(x, g.E)
        assert s == t
    # both stop at ||r|| <= 1e-11 ||b||; A >= 1, so each error is at most that relative to ||b||,
    # and ||x|| is no more than a few times below ||b||
    x1, a, rc1 = run_step(grids, rtol=1e-11, krylov=1, fmg=0, **kw)
    x0, b, rc0 = run_step(grids, rtol=1e-11, krylov=0, fmg=0, **kw)
    assert rc1 == 0 and rc0 == 0
    for x, y in zip(x1, x0):
        assert rel_l2(x, y) <= 1e-10
