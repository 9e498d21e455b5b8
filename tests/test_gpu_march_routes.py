"""The march kernel on grids that the size rule sends there: strips at walls, a last strip
of one column, totals, ensembles of uneven instances and stage saving, in both
types.  Every case first asserts, by the host's rule, that it steps by strips."""

import numpy as np
import pytest
import torch

from paper_2601_02540_amd import workloads as W
from paper_2601_02540_amd.binding import Batch
from gpu_util import dev, solver
from march_plan import batch_plan, plan

pytestmark = pytest.mark.gpu

PER, REF = W.PERIODIC, W.REFLECTING
F32, F64 = torch.float32, torch.float64


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def problem(nx, ny, bx, by, seed):
    g = W.Grid(nx, ny, 0.0, 0.1 * nx, 0.0, 0.1 * ny, bx, by, 9.81, 500.0)
    q, b = W.random_state(g, seed, 0.05)
    q[1:4] *= 0.1
    return g, q, b


def on_strips(g, dtype):
    return plan(g.nx, g.ny, g.bc_x, g.bc_y, dtype.itemsize, cus()) is not None


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("nx,ny,bx,by,steps", [
    (56 * 36 + 1, 2100, REF, REF, 3),
    (56 * 36 + 1, 1700, PER, PER, 1),
    (56 * 26 + 55, 1409, REF, PER, 2),
    (1600, 1604, PER, REF, 5),
    (8200, 300, REF, REF, 1),
])
def test_strips_equal_stage_path(nx, ny, bx, by, steps, dtype):
    g, q, b = problem(nx, ny, bx, by, nx + ny)
    assert on_strips(g, dtype)
    out = []
    for path in ("fused", "stages"):
        s = solver(g, dtype)
        s.set_step_path(path)
        s.set_bathymetry(dev(b, dtype))
        qd = dev(q, dtype)
        s.step(qd, s.cfl_dt(qd, 0.25), steps)
        s.check()
        out.append(qd)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("bx,by", [(PER, PER), (REF, REF), (PER, REF)])
def test_totals_on_strips(bx, by, dtype):
    """The series within rounding of the totals pass (compensated sums in another order:
    a few units in the last place), the state to the bit."""
    g, q, b = problem(56 * 26 + 55, 1409, bx, by, 8)
    assert on_strips(g, dtype)
    s = solver(g, dtype)
    s.set_bathymetry(dev(b, dtype))
    qd, ref = dev(q, dtype), dev(q, dtype)
    dt = s.cfl_dt(qd, 0.25)
    series = s.step_totals(qd, dt, 3).cpu().numpy()
    for k in range(3):
        s.step(ref, dt, 1)
        assert np.allclose(series[k], s.mass_energy(ref), rtol=1e-14, atol=0.0)
    assert torch.equal(qd, ref)


@pytest.mark.parametrize("steps", [1, 3, 10])
def test_f32_ensemble_on_strips(steps):
    cases = [problem(nx, ny, bx, bx, nx) for nx, ny, bx in ((1400, 1801, REF), (57, 64, PER), (1513, 1200, PER),
                                                            (120, 9, REF), (112, 333, REF), (6, 5, PER))]
    assert batch_plan([(g.nx, g.ny, g.bc_y) for g, _, _ in cases], 4, cus()) is not None
    batch = Batch([c[0] for c in cases], F32)
    qs = [dev(q, F32) for _, q, _ in cases]
    for k, (_, _, b) in enumerate(cases):
        batch.set_bathymetry(k, dev(b, F32))
    batch.set_states(qs)
    dts = batch.cfl_dt(0.25)
    batch.step(dts, steps)
    assert batch.check() == -1
    for (g, q, b), got, dt in zip(cases, qs, dts):
        s = solver(g, F32)
        s.set_step_path("stages")
        s.set_bathymetry(dev(b, F32))
        ref = dev(q, F32)
        s.step(ref, dt, steps)
        assert torch.equal(got, ref), (g.nx, g.ny)


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("nx,ny,bx,by", [
    (56 * 26 + 55, 1409, PER, PER),
    (56 * 26 + 55, 1409, REF, PER),
    (1500, 900, REF, REF),
    (56 * 36 + 1, 1700, REF, REF),
    (1600, 1604, PER, REF),
])
def test_stage_saving_on_strips(nx, ny, bx, by, dtype):
    """A step's VJP from stages saved on strips and on 32 x 16 tiles (the reverse kernels are the same)."""
    g, q, b = problem(nx, ny, bx, by, 5)
    assert on_strips(g, dtype)
    rng = np.random.default_rng(6)
    a, bb0 = rng.standard_normal(q.shape), rng.standard_normal(b.shape)
    out = []
    for ty in (None, 16):
        s = solver(g, dtype)
        if ty:
            s.set_tile_y(ty)
        s.set_bathymetry(dev(b, dtype))
        qd, qb, bb = dev(q, dtype), dev(a, dtype), dev(bb0, dtype)
        s.step_vjp(qd, s.cfl_dt(qd, 0.25), qb, bb)
        out.append((qb, bb))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert torch.isfinite(out[0][0]).all()
