"""Which 3D plans march on level 0: with two sweeps each way from zero (conjugate gradients) those of
more tiles than compute units; where single sweeps are needed (plain V-cycles from the iterate, other
sweep counts) those of more than four rounds of tiles.  The steps agree with the launches per colour
on every bit either way."""
import numpy as np
import pytest

import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kw,levels", [((64, 64, 64), {}, 1), ((64, 64, 64), dict(krylov=0), 0),
                                             ((64, 64, 64), dict(nu1=4, nu2=4), 0), ((80, 72, 80), dict(krylov=0), 0),
                                             ((64, 64, 64), dict(nu1=1, nu2=1), 0), ((96, 96, 96), dict(krylov=0), 1),
                                             ((64, 64, 64), dict(krylov=0, fused3_levels=1), 1)])
def test_level_0_marches_where_its_launches_fill_the_card(shape, kw, levels):
    plan = fld.Plan([shape], **kw)
    assert plan.tuning()["fused3_levels"] == levels
    plan.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kw", [dict(krylov=0), dict(krylov=0, fmg=0), dict(nu1=4, nu2=4), dict(nu1=3, nu2=3)])
def test_same_bits_as_launches_per_colour(kw, precision):
    g = W.random_grid((64, 64, 72), 99500, dt=2e-3)
    (a,), (sa,), _ = run_step([g], precision=precision, **kw)
    (b,), (sb,), _ = run_step([g], precision=precision, fused=0, **kw)
    assert np.array_equal(a, b) and sa["cycles"] == sb["cycles"]
