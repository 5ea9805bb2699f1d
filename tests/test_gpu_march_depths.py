"""The two-sweep 3D march at the plane depths that larger plans choose, with windows that end inside
the level on every axis, and r . z formed in it.

Depths by the rule of fewest block steps on 256 compute units: 32 planes (42 windows of a column of
grids of 40 x 24 x 1344 cells; 136^3), 64 planes (160^3 beside 64^3).  Where the CG sums come from
the same kernels (up to 2048 tiles of level 0, or FP32 V-cycles) the step has the bits of the
launches per colour.  Where r . z comes from the march its order differs: the scalars by a few eps,
and the iterate by no more than their number of cycles times that, far below what a wrong sweep
does to it (its correction, rtol)."""
import numpy as np
import pytest

import workloads as W
from oracle import dirichlet as OD
from oracle import fld as OF
from tests.gpu_common import rel_l2, run_step

pytestmark = pytest.mark.gpu


def both(shapes, **kw):
    # (40 x 24 x 1344 does not converge in 50 cycles with either)
    gs = [W.random_grid(s, 99700 + 7 * i, dt=2e-3) for i, s in enumerate(shapes)]
    a = run_step(gs, **kw)
    b = run_step(gs, fused=0, **kw)
    assert a[2] == b[2] and [s["cycles"] for s in a[1]] == [s["cycles"] for s in b[1]]
    return gs, a[0], b[0], a[1]


@pytest.mark.parametrize("fmg", [0, 1])
@pytest.mark.parametrize("shapes,precision", [([(1344, 24, 40)], 0), ([(1344, 24, 40)], 1), ([(136, 136, 136)], 1),
                                              ([(160, 160, 160), (64, 64, 64)], 1)])
def test_bits_of_the_launches_per_colour(shapes, precision, fmg):
    _, xa, xb, _ = both(shapes, precision=precision, fmg=fmg)
    for x, y in zip(xa, xb):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("shapes", [[(144, 136, 152)], [(160, 160, 160), (64, 64, 64)], [(144, 136, 152), (184, 200, 208)]])
def test_r_z_from_the_march(shapes):
    gs, xa, xb, st = both(shapes, precision=0)
    assert all(s["status"] == 0 for s in st)
    for x, y, s in zip(xa, xb, st):
        assert rel_l2(x, y) <= 64 * s["cycles"] * np.finfo(np.float64).eps
    # the first grid's residual with the oracle's operator: the target, and eps in each coefficient and sum
    g, x = gs[0], xa[0].ravel()
    R = np.sqrt(sum(v * v for v in OD.gradient4_general(g.E, g.h))) / (g.kappa_rho * g.E)
    A = OD.assemble_general(OD.face_weights_general(OF.flux_limiter(R, "lp") / g.kappa_rho, g.dt, g.h)).tocsr()
    b = g.E.ravel()
    rounding = 16 * np.finfo(np.float64).eps * np.linalg.norm(abs(A) @ abs(x))
    assert np.linalg.norm(b - A @ x) <= 1e-10 * np.linalg.norm(b) + rounding
