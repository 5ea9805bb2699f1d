"""Which 3D plans march on level 0: with two sweeps each way from zero (conjugate gradients) those of
more tiles than compute units; where single sweeps are needed (plain V-cycles from the iterate, other
sweep counts) those of more than four rounds of tiles and of windows enough.  The steps agree with the launches per colour
on every bit either way."""
import numpy as np
import pytest

import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kw,levels", [((64, 64, 64), {}, 1), ((64, 64, 64), dict(krylov=0), 0),
                                             ((64, 64, 64), dict(nu1=4, nu2=4), 0), ((80, 72, 80), dict(krylov=0), 0),
                                             ((64, 64, 64), dict(nu1=1, nu2=1), 0), ((100, 100, 100), dict(krylov=0), 0),
                                             ((128, 128, 128), dict(krylov=0), 1), ((100, 100, 100), {}, 1),
                                             ((64, 64, 64), dict(krylov=0, fused3_levels=1), 1)])
def test_level_0_marches_where_its_launches_fill_the_card(shape, kw, levels):
    plan = fld.Plan([shape], **kw)
    assert min(1, plan.tuning()["fused3_levels"]) == levels
    plan.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kw", [dict(krylov=0), dict(krylov=0, fmg=0), dict(nu1=4, nu2=4), dict(nu1=3, nu2=3)])
def test_same_bits_as_launches_per_colour(kw, precision):
    g = W.random_grid((64, 64, 72), 99500, dt=2e-3)
    (a,), (sa,), _ = run_step([g], precision=precision, **kw)
    (b,), (sb,), _ = run_step([g], precision=precision, fused=0, **kw)
    assert np.array_equal(a, b) and sa["cycles"] == sb["cycles"]


# r . z of a large grid comes from the two-sweep march, whose plane depth is the plan's: 64 beside
# the other grid in the first and the last case, 8 in place of 32 in the second; the direction
# pass' depth is the same alone and beside it
@pytest.mark.parametrize("shape,other", [((160, 160, 160), (64, 64, 64)), ((136, 136, 136), (96, 96, 96)),
                                         ((136, 136, 136), (208, 208, 208))])
def test_sums_do_not_depend_on_the_depth_of_the_windows(shape, other):
    a, b = W.random_grid(shape, 99600, dt=2e-3), W.random_grid(other, 99601, dt=1e-3)
    (xa,), (sa,), _ = run_step([a])
    xb, sb, _ = run_step([a, b])
    assert sa["cycles"] == sb[0]["cycles"] and sa["rel_residual"] == sb[0]["rel_residual"]
    assert np.array_equal(xa, xb[0])


def test_profile_of_the_march():
    plan = fld.Plan([(64, 64, 64)])
    ms, cells = plan.profile(fld.FLD_KERNEL_MARCH3, 0, 5)
    assert ms > 0 and cells == 64 ** 3
    with pytest.raises(fld.FLDError):
        plan.profile(fld.FLD_KERNEL_MARCH3, 1, 5)              # a level of tiles
    plan.close()
    plan = fld.Plan([(64, 64, 64)], krylov=0)
    with pytest.raises(fld.FLDError):
        plan.profile(fld.FLD_KERNEL_MARCH3, 0, 5)
    plan.close()
