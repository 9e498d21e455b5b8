"""Health flag of the small-grid kernel's two-step launches.

Four steps are two launches of two steps.  The states (from the oracle) stay
positive through the steps before the one that fails, the second of a launch; with
four steps in all nothing after it could raise the flag."""

import numpy as np
import pytest
import torch

import oracle
from paper_2601_02540_amd import workloads as W
from paper_2601_02540_amd.binding import SgnError
from gpu_util import dev, solver

pytestmark = pytest.mark.gpu

NONPOS_DEPTH = -5


def depths(g, q, b, dt, steps):
    out = []
    for _ in range(steps):
        q = oracle.rk4(g, q, b, dt, 1)
        out.append(q[0].min() if np.isfinite(q).all() else np.nan)
    return out


# (seed, velocities' factor, CFL, steps, the first step that fails)
@pytest.mark.parametrize("seed,amp,cfl,steps,bad", [
    (1, 4.0, 2.0, 4, 4),
    (3, 1.0, 2.0, 4, 4),
    (3, 4.0, 2.0, 4, 4),
    (4, 4.0, 2.0, 6, 4),
    (1, 4.0, 2.0, 3, 0),
    (0, 1.0, 0.5, 4, 0),
])
def test_failure_in_a_launch_of_two_steps(seed, amp, cfl, steps, bad):
    g = W.Grid(24, 24, 0.0, 2.4, 0.0, 2.4, W.PERIODIC, W.PERIODIC, 9.81, 500.0)
    q, b = W.random_state(g, seed, 0.05)
    q[1:4] *= amp
    dt = oracle.cfl_dt(g, q, cfl)
    h = depths(g, q, b, dt, bad if bad else steps)
    assert min(h[:-1]) > 1e-2 and (h[-1] < -1e-2 if bad else h[-1] > 1e-2), h
    s = solver(g)
    s.set_bathymetry(dev(b))
    qd = dev(q)
    s.step(qd, dt, steps)
    if not bad:
        s.check()
        assert torch.isfinite(qd).all() and bool((qd[0] > 0).all())
        return
    with pytest.raises(SgnError) as e:
        s.check()
    if steps == bad:  # finite up to here
        assert e.value.status == NONPOS_DEPTH
    s.check()  # reported once
