"""The small-grid step kernel (two steps per launch on 8 x 8 tiles) against the
four-stage path, to the bit: axes shorter than its halo, ragged tiles, every
boundary pair, and the step counts that its launches split differently."""

import pytest
import torch

from paper_2601_02540_amd import workloads as W
from gpu_util import dev, solver

pytestmark = pytest.mark.gpu

PER, REF = W.PERIODIC, W.REFLECTING


@pytest.mark.parametrize("nx,ny,bx,by,dtype", [
    (4, 4, PER, PER, torch.float64),
    (5, 9, REF, PER, torch.float64),
    (8, 6, PER, REF, torch.float32),
    (64, 64, PER, PER, torch.float64),
    (33, 100, REF, REF, torch.float64),
    (97, 17, REF, REF, torch.float32),
    (256, 250, PER, REF, torch.float64),
])
def test_small_grid_steps_equal_stage_path(nx, ny, bx, by, dtype):
    g = W.Grid(nx, ny, 0.0, 0.1 * nx, 0.0, 0.1 * ny, bx, by, 9.81, 500.0)
    q, b = W.random_state(g, nx + ny, 0.05)
    q[1:4] *= 0.1
    for steps in (1, 2, 3, 4, 5, 6, 7, 8, 9, 18):
        out = []
        for path in ("fused", "stages"):
            s = solver(g, dtype)
            s.set_step_path(path)
            s.set_bathymetry(dev(b, dtype))
            qd = dev(q, dtype)
            s.step(qd, s.cfl_dt(qd, 0.2), steps)
            s.check()
            out.append(qd)
        assert torch.equal(out[0], out[1]), steps


def test_small_grid_health_flag():
    """A depth that turns non-positive in either of a launch's two steps is reported."""
    g = W.Grid(24, 24, 0.0, 1.0, 0.0, 1.0, PER, PER, 9.81, 500.0)
    q, b = W.random_state(g, 1, 0.05)
    for steps in (1, 2):
        s = solver(g)
        s.set_bathymetry(dev(b))
        qd = dev(q)
        s.step(qd, 60.0 * s.cfl_dt(qd, 0.5), steps)
        with pytest.raises(Exception):
            s.check()
