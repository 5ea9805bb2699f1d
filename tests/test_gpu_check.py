"""The check at the end of a step (norm and output in one pass): with a target below what FP64
can reach, grids come back from it to iterate again, next to grids that pass it."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import rel_l2, run_step

pytestmark = pytest.mark.gpu

SHAPES = [(24, 17), (65, 64), (130, 97), (12, 9, 10), (20, 33, 17)]


@pytest.mark.parametrize("precision", [0, 1])
def test_grids_sent_back_by_the_check(precision):
    grids = [W.random_grid(s, 93000 + i, dt=1e-3) for i, s in enumerate(SHAPES)]
    good, _, rc = run_step(grids, precision=precision, rtol=1e-12)
    assert rc == 0
    for rtol in (1e-15, 3e-16, 1e-16):
        xs, st, _ = run_step(grids, precision=precision, rtol=rtol)
        for x, y, s in zip(xs, good, st):
            # a step says it converged only with a true residual within its target
            assert (s["status"] == 0) == (s["rel_residual"] <= rtol)
            # either way the iterate is within both targets (A >= 1; ||b|| is a few ||x|| at most),
            # and every grid's output is written
            assert rel_l2(x, y) <= 1e-10


def test_output_of_a_step_that_stops_at_once():
    # rtol met by the start: E_out = E_in, for a grid beside one with invalid input too
    grids = [W.random_grid(s, 93100 + i, dt=1e-9) for i, s in enumerate(SHAPES[:3])]
    for fmg in (0, 1):
        xs, st, rc = run_step(grids, rtol=0.5, fmg=fmg)
        assert rc == 0
        for x, g in zip(xs, grids):
            assert np.array_equal(x, g.E)
    grids[1].kappa_rho[3, 3] = np.nan
    xs, st, rc = run_step(grids, rtol=0.5)
    assert rc != 0 and st[0]["status"] == 0 and st[1]["status"] != 0
    for x, g in zip(xs, grids):
        assert np.array_equal(x, g.E)
