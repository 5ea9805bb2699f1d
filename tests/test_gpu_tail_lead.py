"""Levels of more than 2048 cells that head an LDS tail: grids that live in it whole, and the first
tail level of plans whose levels above sweep per colour.

The route shows in the launches of a multigrid pass: 1 for a whole grid; 11 with one level above
(four half sweeps and the restriction, the tail, the prolongation and four half sweeps).  The step's
residual is taken with the oracle's operator: at most rtol ||b||, and what a relative error of eps
in each coefficient and sum makes of it."""
import numpy as np
import pytest
import torch

import paper_2104_03968_amd as fld
import workloads as W
from oracle import dirichlet as OD
from tests.gpu_common import dev, run_step

pytestmark = pytest.mark.gpu

CODE = {"zero_flux": fld.FLD_BC_ZERO_FLUX, "periodic": fld.FLD_BC_PERIODIC, "dirichlet": fld.FLD_BC_DIRICHLET,
        "continuous": fld.FLD_BC_CONTINUOUS}
VALUES = [1.5, 0.5, 2.0, 1.0, 0.25, 0.75]
RTOL = 1e-10


def kinds_of(name, dim):
    return {"box": ["periodic"] * (2 * dim - 2) + ["dirichlet"] * 2}.get(name, [name] * (2 * dim))


def step_and_launches(shape, bc, **kw):
    dim = len(shape)
    g = W.random_grid(shape, 98000 + sum(shape), dt=1e-3)
    kinds = kinds_of(bc, dim)
    values = [v if k == "dirichlet" else 0.0 for v, k in zip(VALUES, kinds)]
    _, info = OD.diffusion_step_general(g.E, g.kappa_rho, g.dt, g.h, kinds, values, tol=1e-3)
    A, b = info.extra["A"], info.extra["b"].ravel()
    pad = 6 - 2 * dim
    plan = fld.Plan([shape], h=[g.h], rtol=RTOL, max_cycles=100, bc=[CODE[k] for k in kinds] + [CODE["zero_flux"]] * pad,
                    bc_value=values + [0.0] * pad, **kw)
    launches = plan.cycle_bytes(fld.FLD_CYCLE_MG)[1]
    E, out = dev(g.E), torch.empty(shape, dtype=torch.float64, device="cuda")
    plan.step([E], [dev(g.kappa_rho)], [out], [g.dt])
    plan.close()
    x = out.cpu().numpy().ravel()
    rounding = 16 * np.finfo(np.float64).eps * np.linalg.norm(abs(A) @ abs(x))
    assert np.linalg.norm(b - A @ x) <= RTOL * np.linalg.norm(b) + rounding
    return launches


# the smallest above 2048 cells, the largest that the LDS holds; a single level and several below
@pytest.mark.parametrize("fmg", [0, 1])
@pytest.mark.parametrize("shape,precision", [((16, 12, 12), 0), ((14, 14, 14), 0), ((26, 10, 8), 0), ((4, 4, 130), 0),
                                             ((12, 16, 12), 1), ((16, 16, 16), 1), ((18, 18, 18), 1)])
@pytest.mark.parametrize("bc", ["zero_flux", "periodic", "box"])
def test_whole_3d_grids(shape, precision, bc, fmg):
    # (with couplings 18^3 is past the LDS: a pass of tiles down and one up above the tail)
    launches = 3 if bc == "box" and shape == (18, 18, 18) else 1
    assert step_and_launches(shape, bc, precision=precision, fmg=fmg) == launches


# whole 2D grids with fused passes have no lead level
@pytest.mark.parametrize("shape", [(46, 46), (64, 64), (4, 1024), (1024, 4), (8, 512), (52, 78)])
@pytest.mark.parametrize("precision", [0, 1])
def test_whole_2d_grids(shape, precision):
    assert step_and_launches(shape, "zero_flux", precision=precision) == 3


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("bc", ["periodic", "box", "continuous"])
@pytest.mark.parametrize("shape,launches", [((52, 52), 1), ((46, 48), 1), ((100, 104), 11), ((14, 14, 14), 1), ((28, 24, 28), 11)])
def test_levels_swept_per_colour(shape, launches, bc, precision):
    assert step_and_launches(shape, bc, precision=precision, krylov=0) == launches


# sweep counts that the fused passes do not take
@pytest.mark.parametrize("shape,precision,nu1,nu2,launches", [((100, 104), 0, 4, 4, 19), ((128, 128), 1, 4, 4, 19),
                                                              ((32, 32, 32), 1, 1, 2, 9), ((28, 24, 28), 0, 1, 2, 9)])
def test_sweep_counts_of_launches_per_colour(shape, precision, nu1, nu2, launches):
    assert step_and_launches(shape, "zero_flux", precision=precision, nu1=nu1, nu2=nu2, krylov=0) == launches


# the choice does not depend on the fused option, which changes no bit
@pytest.mark.parametrize("shape,precision", [((64, 64), 0), ((64, 64), 1), ((128, 128), 1), ((16, 16, 16), 1), ((32, 24, 32), 0)])
def test_same_bits_without_fused_passes(shape, precision):
    g = W.random_grid(shape, 99000 + sum(shape), dt=1e-3)
    for krylov in (0, 1):
        (a,), (sa,), _ = run_step([g], precision=precision, krylov=krylov)
        (b,), (sb,), _ = run_step([g], precision=precision, krylov=krylov, fused=0)
        assert np.array_equal(a, b) and sa["cycles"] == sb["cycles"]


# a lead level beside them sends every grid's tail to another instantiation of the kernel
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["zero_flux", "periodic"])
def test_grids_beside_a_lead_level_keep_their_bits(kind, precision):
    shapes = [(8, 8, 8), (12, 12, 12), (24, 24, 24), (11, 11, 11), (40, 24, 32), (13, 12, 13), (3, 5, 7)]
    kw = dict(precision=precision, bc=[CODE[kind]] * 6)
    gs = [W.random_grid(s, 99100 + i, dt=2e-3) for i, s in enumerate(shapes)]
    xb, sb, _ = run_step(gs + [W.random_grid((14, 14, 14), 99190, dt=2e-3)], **kw)
    for i, g in enumerate(gs):
        (xa,), (sa,), _ = run_step([g], **kw)
        assert np.array_equal(xa, xb[i]) and sa["cycles"] == sb[i]["cycles"], shapes[i]
