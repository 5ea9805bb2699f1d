"""The LDS tail: grids that live in it whole, at the sizes where its levels change hands.

The first level is swept by the workgroup (one or two cells of a colour a thread), the second too
where it has more than a wavefront's cells, every level below by a wavefront; the coarsest is
solved by conjugate gradients on one colour, by the workgroup or a wavefront, or on all cells where
an odd periodic axis does not split red-black.  Each step meets the FP64 oracle at the residual
bound: ||x - x*|| <= q_b rtol ||x*|| (A is SPD with lambda_min >= 1), with rtol = 1e-10 / q_b the
relative error is at most 1e-10."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import dev, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [
    (32, 32), (64, 32), (44, 46),            # two cells of a colour a thread; 22 x 23: coarsest on the workgroup
    (36, 28), (24, 20), (16, 16), (8, 8),    # 18 x 14: 126 of a colour, one wavefront
    (15, 15), (45, 25), (31, 33), (3, 85), (2, 2), (5, 2), (2, 341),   # one level; thin and odd rows
    (12, 12, 12), (8, 8, 8), (10, 14, 14), (4, 4, 4), (11, 11, 11), (3, 3, 3), (16, 12, 8), (2, 2, 2), (20, 10, 10),
]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_grids_meet_the_oracle(shape, precision):
    g = W.random_grid(shape, 81000 + sum(shape), dt=5e-3)
    x_or = O.diffusion_step(g.E, g.kappa_rho, g.dt, g.h)[0]
    plan = fld.Plan([shape], h=[g.h], precision=precision, rtol=1e-10 / O.q_b(g.E))
    E, out = dev(g.E), torch.empty(shape, dtype=torch.float64, device="cuda")
    plan.step([E], [dev(g.kappa_rho)], [out], [g.dt])
    assert rel_l2(out.cpu().numpy(), x_or) <= 1e-10
    plan.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", [(24, 20), (36, 12), (15, 15), (24, 12), (12, 8, 20), (9, 9, 9), (6, 10, 14)])
def test_small_periodic_and_dirichlet_grids_meet_the_oracle(shape, precision):
    P, D = "periodic", "dirichlet"
    kinds = [P, P, P, P] if len(shape) == 2 else [P, P, P, P, D, D]
    values = [0.0] * 4 if len(shape) == 2 else [0.0] * 4 + [1.5, 0.5]
    g = W.random_grid(shape, 82000 + sum(shape), dt=5e-3)
    x_or, info = O.diffusion_step_general(g.E, g.kappa_rho, g.dt, g.h, kinds, values, method="direct")
    b = info.extra["b"]
    rtol = 1e-10 * np.linalg.norm(x_or) / np.linalg.norm(b) / max(1.0, O.q_b(b))
    code = {P: fld.FLD_BC_PERIODIC, D: fld.FLD_BC_DIRICHLET}
    pad = [fld.FLD_BC_ZERO_FLUX] * (6 - len(kinds))
    plan = fld.Plan([shape], h=[g.h], precision=precision, rtol=rtol, bc=[code[k] for k in kinds] + pad,
                    bc_value=values + [0.0] * (6 - len(values)))
    E, out = dev(g.E), torch.empty(shape, dtype=torch.float64, device="cuda")
    plan.step([E], [dev(g.kappa_rho)], [out], [g.dt])
    assert rel_l2(out.cpu().numpy(), x_or) <= 1e-10
    plan.close()
