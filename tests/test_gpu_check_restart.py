"""Grids that conjugate gradients stop on their recursive residual and the check at the end of a step
sends back: they iterate again from a residual that is formed anew, and converge.

That a grid was sent back shows in the recursive residual, which a step with an unreachable target
reports after every number of cycles (the arithmetic does not know the target): it meets the target
after `k` cycles, and the step takes more.  The request server checks with a pass that forms that
residual in any case, so it must give the same bits in the same number of cycles."""
import numpy as np
import pytest

import paper_2104_03968_amd as fld
import workloads as W
from tests.gpu_common import dev, run_step

pytestmark = pytest.mark.gpu

CASES = [((200, 200), 0.1, 3e-14), ((200, 200), 0.01, 1e-14), ((65, 64), 0.01, 1e-15), ((130, 97), 0.1, 1e-14),
         ((64, 64, 40), 0.1, 1e-14), ((64, 64, 40), 0.01, 1e-15)]


def served(g, precision, rtol):
    srv = fld.Server(64 << 20, precision=precision, rtol=rtol, max_cycles=60)
    try:
        E, kr = dev(g.E), dev(g.kappa_rho)                     # read at admission
        t = srv.submit(E, kr, g.dt, h=g.h)
        rc, res = srv.wait(t)
        return rc, res.stats.cycles, srv.result_tensor(res, g.E.shape).cpu().numpy()
    finally:
        srv.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape,dt,rtol", CASES)
def test_a_grid_sent_back_converges(shape, dt, rtol, precision):
    g = W.random_grid(shape, 93500 + sum(shape), dt=dt)
    kw = dict(precision=precision, fmg=0)
    (x,), (st,), rc = run_step([g], rtol=rtol, max_cycles=60, **kw)
    stop = next(k for k in range(1, 60)
                if run_step([g], rtol=1e-30, max_cycles=k, **kw)[1][0]["rel_residual"] <= rtol)
    assert st["cycles"] > stop
    assert rc == 0 and st["status"] == 0 and st["rel_residual"] <= rtol
    rc, cycles, y = served(g, precision, rtol)
    assert rc == 0 and cycles == st["cycles"]
    assert np.array_equal(x, y)
    # beside a grid that passes at once, and one that is still iterating then
    others = [W.random_grid((24, 17) if len(shape) == 2 else (12, 9, 10), 93700, dt=1e-6),
              W.random_grid((300, 260) if len(shape) == 2 else (72, 64, 48), 93701, dt=0.3)]
    xs, sts, _ = run_step([others[0], g, others[1]], rtol=rtol, max_cycles=60, **kw)
    assert sts[1]["status"] == 0 and sts[1]["cycles"] == st["cycles"]
    assert np.array_equal(xs[1], x)
