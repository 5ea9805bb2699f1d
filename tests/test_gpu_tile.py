"""3D passes of several red-black sweeps per launch: small levels' tiles in LDS and registers, and
the two-sweep z-march of large levels.

They use the operand order of the per-colour kernels, so a plan that runs them and one that
sweeps per colour (fused = 0) agree on every bit, on every level size around the tile's
interior (4, 8 and 10 cells a side in 3D, 52, 56 and 58 in 2D), at every sweep count, from zero
and from an iterate, and with every kind of boundary that conjugate gradients solve."""
import numpy as np
import pytest
import torch

import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import dev

pytestmark = pytest.mark.gpu

Z, P, D = fld.FLD_BC_ZERO_FLUX, fld.FLD_BC_PERIODIC, fld.FLD_BC_DIRICHLET
# levels of 1, 2 and 3 tiles a side, one cell pair below, at and above the interiors' multiples
SHAPES3 = [(16, 16, 16), (36, 20, 44), (18, 34, 62), (24, 40, 80), (66, 22, 28)]
SHAPES2 = [(112, 56), (208, 116), (106, 174), (120, 240)]


def step(shapes, drop_optional=False, **kw):
    gs = [W.random_grid(s, 71000 + 7 * i, dt=3e-3) for i, s in enumerate(shapes)]
    h = [(1.0 / max(s),) * len(s) for s in shapes]
    opts = fld.fld_opts_default(**kw)
    grids = [fld.make_grid(tuple(reversed(s)), hh) for s, hh in zip(shapes, h)]
    plan = fld.fld_plan_create(grids, opts)
    try:
        need = fld.fld_plan_workspace_bytes(plan)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        fld.fld_plan_bind_workspace(plan, ws.data_ptr(), need - (256 if drop_optional else 0))
        E, K = [dev(g.E) for g in gs], [dev(g.kappa_rho) for g in gs]
        out = [torch.empty_like(e) for e in E]
        launches = fld.fld_plan_cycle_bytes(plan, fld.FLD_CYCLE_MG)[1]
        rc, st = fld.fld_step(plan, E, K, out, [3e-3] * len(gs), check=False)
        torch.cuda.synchronize()
        return rc, [(s["status"], s["cycles"]) for s in st], [o.cpu().numpy() for o in out], launches
    finally:
        fld.fld_plan_destroy(plan)


def same(a, b, fewer=True):
    assert a[0] == b[0] and a[1] == b[1]
    for i, (x, y) in enumerate(zip(a[2], b[2])):
        assert np.array_equal(x, y), (i, np.abs(x - y).max())
    assert (a[3] < b[3]) == fewer, (a[3], b[3])


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nu_coarse", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("nu", [1, 2, 3])
def test_three_dimensional_levels_bitwise(nu, nu_coarse, precision):
    kw = dict(nu1=nu, nu2=nu, nu_coarse=nu_coarse, precision=precision)
    same(step(SHAPES3, **kw), step(SHAPES3, fused=0, **kw))


# windows of 32 x 16 columns and a halo of four: one pair below, at and above their multiples
SHAPES_MARCH = [(8, 16, 32), (24, 18, 34), (40, 30, 62), (12, 34, 66), (76, 46, 30)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nu,nu_coarse,fmg", [(2, 2, 1), (2, 3, 0), (3, 2, 1), (4, 5, 0)])
def test_two_sweep_march_bitwise(nu, nu_coarse, fmg, precision):
    kw = dict(nu1=nu, nu2=nu, nu_coarse=nu_coarse, precision=precision, fmg=fmg)
    same(step(SHAPES_MARCH, fused3_levels=9, **kw), step(SHAPES_MARCH, fused=0, **kw))


@pytest.mark.parametrize("krylov,fmg,precision", [(0, 1, 0), (0, 0, 0), (0, 1, 1), (1, 0, 0), (1, 0, 1)])
def test_starts_from_zero_and_from_an_iterate_bitwise(krylov, fmg, precision):
    kw = dict(krylov=krylov, fmg=fmg, fmg_depths=0, precision=precision, max_cycles=30)
    same(step(SHAPES3, **kw), step(SHAPES3, fused=0, **kw))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shapes", [SHAPES3, SHAPES2])
@pytest.mark.parametrize("kinds", [(P, P, P), (D, D, D), (P, P, D), (D, P, Z)])
def test_boundary_kinds_bitwise(kinds, shapes, precision):
    bc = [k for k in kinds for _ in (0, 1)]
    kw = dict(bc=bc, bc_value=[0.5, 1.5, 0.0, 2.0, 1.0, 0.25], precision=precision)
    a = step(shapes, **kw)
    same(a, step(shapes, fused=0, **kw))
    # a workspace without the optional part sweeps per colour, to the same bits
    same(step(shapes, drop_optional=True, **kw), a, fewer=False)
