"""The march kernel (one wave per strip of 56 columns, large grids) against the
four-stage path: every step path forms the same bits, so the states are compared
exactly.  Sizes sit at the edges of its cut: a last strip of one column, of 55 and
a full one, runs of rows that do not divide the height, all four boundary pairs,
step counts that end the buffer rotation each way."""

import numpy as np
import pytest
import torch

from paper_2601_02540_amd import workloads as W
from paper_2601_02540_amd.binding import Batch
from gpu_util import check_windows, dev, host, solver

pytestmark = pytest.mark.gpu

PER, REF = W.PERIODIC, W.REFLECTING


def problem(nx, ny, bx, by, seed):
    g = W.Grid(nx, ny, 0.0, 0.1 * nx, 0.0, 0.1 * ny, bx, by, 9.81, 500.0)
    q, b = W.random_state(g, seed, 0.05)
    q[1:4] *= 0.1  # a stable start: random depths, small velocities
    return g, q, b


@pytest.mark.parametrize("nx,ny,bx,by,dtype,steps", [
    (56 * 19 + 1, 1000, PER, PER, torch.float64, 1),
    (56 * 19, 1003, REF, REF, torch.float64, 3),
    (56 * 18 + 55, 997, REF, PER, torch.float64, 2),
    (56 * 18 + 29, 1031, PER, REF, torch.float64, 5),
    (56 * 19 + 1, 1000, REF, REF, torch.float32, 3),
    (56 * 18 + 55, 1009, PER, PER, torch.float32, 4),
    (4096 + 3, 261, PER, REF, torch.float32, 2),
    (300, 3600, REF, PER, torch.float64, 1),
])
def test_march_equals_stage_path(nx, ny, bx, by, dtype, steps):
    g, q, b = problem(nx, ny, bx, by, nx + ny)
    out = []
    for path in ("fused", "stages"):
        s = solver(g, dtype)
        s.set_step_path(path)
        s.set_bathymetry(dev(b, dtype))
        qd = dev(q, dtype)
        dt = s.cfl_dt(qd, 0.25)
        s.step(qd, dt, steps)
        s.check()
        out.append(qd)
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_march_batch_and_totals(dtype):
    """Ensemble strips of uneven instances, odd and single steps, and the totals epilogue."""
    cases = [problem(nx, ny, bx, bx, nx) for nx, ny, bx in ((700, 801, REF), (57, 64, PER), (513, 1200, PER),
                                                            (120, 9, REF), (112, 333, REF), (6, 5, PER))]
    for steps in (1, 3, 10):
        batch = Batch([c[0] for c in cases], dtype)
        qs, dts = [], []
        for k, (g, q, b) in enumerate(cases):
            batch.set_bathymetry(k, dev(b, dtype))
            qs.append(dev(q, dtype))
        batch.set_states(qs)
        dts = batch.cfl_dt(0.25)
        batch.step(dts, steps)
        assert batch.check() == -1
        for (g, q, b), got, dt in zip(cases, qs, dts):
            s = solver(g, dtype)
            s.set_step_path("stages")
            s.set_bathymetry(dev(b, dtype))
            ref = dev(q, dtype)
            s.step(ref, dt, steps)
            assert torch.equal(got, ref), (g.nx, g.ny, steps)
    for bx, by in ((PER, PER), (REF, REF)):
        g, q, b = problem(1065, 1000, bx, by, 8)
        s = solver(g, dtype)
        s.set_bathymetry(dev(b, dtype))
        qd, ref = dev(q, dtype), dev(q, dtype)
        dt = s.cfl_dt(qd, 0.25)
        series = s.step_totals(qd, dt, 5).cpu().numpy()
        for k in range(5):
            s.step(ref, dt, 1)
            assert np.allclose(series[k], s.mass_energy(ref), rtol=1e-13, atol=0.0)
        assert torch.equal(qd, ref)


def test_march_against_oracle():
    """Windows of a 1121 x 1024 reflecting run exactly against the oracle."""
    g, q, b = problem(1121, 1024, REF, REF, 2)
    s = solver(g)
    s.set_bathymetry(dev(b))
    qd = dev(q)
    dt = s.cfl_dt(qd, 0.25)
    s.step(qd, dt, 3)
    check_windows(g, q, b, host(qd), dt, 3, [(("wall_lo", 0), ("wall_lo", 0)), (("wall_hi", 0), ("wall_hi", 0)),
                                             (("in", 500), ("in", 540))])
