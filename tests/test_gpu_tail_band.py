"""Single levels of odd nx and up to 2048 cells, whose rows of ceil(nx / 2) cells of a colour do
not fit the LDS tail's threads: counted along the whole level, they are the tail's all the same.

The route shows in the accounted bytes of a multigrid pass: the tail is counted with the faces of a
level and of those below it (a factor 2^d / (2^d - 1)), the direct solve with the level's alone.
Steps meet the FP64 oracle at the residual bound: ||x - x*|| <= q_b rtol ||x*||, with rtol =
1e-10 / q_b at most 1e-10."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import dev, rel_l2

pytestmark = pytest.mark.gpu

# shapes are (nz,) ny, nx: nx odd; in 3D planes of an odd and of an even number of cells
BAND = [(45, 45), (93, 22), (22, 93), (682, 3), (3, 681), (13, 13, 11), (12, 13, 13), (13, 12, 13), (2, 341, 3),
        (341, 2, 3), (227, 3, 3), (4, 102, 5)]
WIDE = [(90, 90), (46, 90)]                                    # a wide level above 45 x 45 and 23 x 45


def plan_and_step(shape, g, **kw):
    plan = fld.Plan([shape], h=[g.h], **kw)
    E, out = dev(g.E), torch.empty(shape, dtype=torch.float64, device="cuda")
    mg = plan.cycle_bytes(fld.FLD_CYCLE_MG)[0]
    plan.step([E], [dev(g.kappa_rho)], [out], [g.dt])
    plan.close()
    return mg, out.cpu().numpy()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", BAND + WIDE)
def test_band_is_the_tails_and_meets_the_oracle(shape, precision):
    g = W.random_grid(shape, 96000 + sum(shape), dt=5e-3)
    x_or = O.diffusion_step(g.E, g.kappa_rho, g.dt, g.h)[0]
    for krylov in (1, 0):
        mg, x = plan_and_step(shape, g, precision=precision, krylov=krylov, rtol=1e-10 / O.q_b(g.E))
        assert rel_l2(x, x_or) <= 1e-10
        if shape in BAND:
            d = len(shape)
            word = 4 if precision else 8
            assert mg == pytest.approx(word * g.E.size * (2 + d * 2 ** d / (2 ** d - 1)), rel=1e-12)


@pytest.mark.parametrize("shape", [(45, 45), (12, 13, 13), (13, 12, 13), (22, 93)])
def test_band_with_held_and_wrapped_faces(shape):
    # held faces split red-black with the flat count; odd periodic axes are solved on all cells,
    # with the operator in LDS
    g = W.random_grid(shape, 97000 + sum(shape), dt=5e-3)
    P, D = "periodic", "dirichlet"
    code = {P: fld.FLD_BC_PERIODIC, D: fld.FLD_BC_DIRICHLET}
    for kinds in ([D] * 6, [P, P, D, D, D, D]):
        kinds = kinds[:2 * len(shape)]
        values = [1.5 if k == D else 0.0 for k in kinds]
        x_or, info = O.diffusion_step_general(g.E, g.kappa_rho, g.dt, g.h, kinds, values, method="direct")
        b = info.extra["b"]
        rtol = 1e-10 * np.linalg.norm(x_or) / np.linalg.norm(b) / max(1.0, O.q_b(b))
        pad = 6 - len(kinds)
        _, x = plan_and_step(shape, g, rtol=rtol, bc=[code[k] for k in kinds] + [fld.FLD_BC_ZERO_FLUX] * pad,
                             bc_value=values + [0.0] * pad)
        assert rel_l2(x, x_or) <= 1e-10
