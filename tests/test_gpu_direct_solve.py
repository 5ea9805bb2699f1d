"""Grids of a single level, too large for the LDS tail or just in it: under conjugate gradients every outer
iteration solves them directly, from zero, to a 1e-6 residual.

The mixed-precision plan makes the same solve in FP32 arrays, so FP64 takes no more outer
iterations than it does; a solve that starts from the previous correction, to 1e-6 of that start's
residual, hardly corrects and takes more.  Steps meet the FP64 oracle at the residual bound:
||x - x*|| <= q_b rtol ||x*|| (A is SPD with lambda_min >= 1)."""
import pytest

import oracle as O
import workloads as W
from tests.gpu_common import rel_l2, run_step

pytestmark = pytest.mark.gpu

# up to and past the 4096 cells whose vectors sit in LDS; beside a grid with fused passes
CASES = [[(47, 47)], [(1025, 3)], [(3, 1025)], [(67, 67)], [(13, 13, 13)], [(257, 3, 3)], [(17, 17, 17)],
         [(1025, 3), (128, 96)], [(257, 3, 3), (72, 64, 64)],
         [(45, 45)], [(13, 12, 13), (72, 64, 64)]]             # single levels at the tail's limit


@pytest.mark.parametrize("shapes", CASES)
def test_direct_solves_start_from_zero(shapes):
    grids = [W.random_grid(s, 95000 + 3 * sum(s), dt=5e-3) for s in shapes]
    x64, st64, rc64 = run_step(grids, precision=0, fmg=0)
    _, st32, rc32 = run_step(grids, precision=1, fmg=0)
    assert rc64 == 0 and rc32 == 0
    assert st64[0]["cycles"] <= st32[0]["cycles"]
    for x, g in zip(x64, grids):
        x_or = O.diffusion_step(g.E, g.kappa_rho, g.dt, g.h)[0]
        assert rel_l2(x, x_or) <= 1e-10 * O.q_b(g.E) * 1.01
