"""Coarse operators of the tails in one launch, a workgroup a grid: a batch whose tails start at
different levels (level 0, one level, none, thin and odd remainders), every level against the
rule applied to the device's finer level at the bound of test_gpu_multigrid (1e-14)."""
import numpy as np
import pytest
import torch

import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import dev
from tests.test_gpu_multigrid import RULES

pytestmark = pytest.mark.gpu

SHAPES = {2: [(2, 2), (4, 64), (64, 4), (64, 64), (180, 100), (33, 20), (130, 96), (256, 6)],
          3: [(2, 2, 2), (4, 4, 64), (16, 24, 20), (32, 32, 32), (17, 20, 23), (40, 8, 12)]}


@pytest.mark.parametrize("coarse_op", ["rediscretised", "galerkin"])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dim", [2, 3])
def test_tail_operators(dim, precision, coarse_op):
    grids = [W.random_grid(s, 94000 + i, dt=2e-3) for i, s in enumerate(SHAPES[dim])]
    plan = fld.Plan([g.E.shape for g in grids], h=[g.h for g in grids], precision=precision, coarse_op=coarse_op)
    E, K = [dev(g.E) for g in grids], [dev(g.kappa_rho) for g in grids]
    plan.coefficients(E, K, [g.dt for g in grids])
    torch.cuda.synchronize()
    for i in range(len(grids)):
        prev = [w.cpu().numpy() for w in plan.level_tensors(i, 0)["w"]]
        for lev in range(1, plan.levels(i)):
            lv = plan.level_tensors(i, lev)
            got = [w.cpu().numpy() for w in lv["w"]]
            for a, want in enumerate(RULES[coarse_op](prev)):
                err = np.abs(got[a] - want) / np.where(want == 0, 1.0, np.abs(want))
                assert err.max() <= 1e-14, (grids[i].E.shape, lev, a, err.max())
                if precision == 1:
                    assert np.array_equal(lv["w32"][a].cpu().numpy(), got[a].astype(np.float32))
            prev = got
    plan.close()
