"""An ensemble of more instances than a launch has block rows: a single step, whose
states are copied back by one launch over all of them."""

import pytest
import torch

from paper_2601_02540_amd import workloads as W
from paper_2601_02540_amd.binding import Batch
from gpu_util import dev, solver

pytestmark = pytest.mark.gpu


def test_single_step_of_more_instances_than_block_rows():
    n = 65600
    g = W.Grid(4, 4, 0.0, 0.4, 0.0, 0.4, W.PERIODIC, W.REFLECTING, 9.81, 500.0)
    q, b = W.random_state(g, 3, 0.05)
    q[1:4] *= 0.1
    q0, bd = dev(q, torch.float32), dev(b, torch.float32)
    factor = 1.0 + 0.1 * torch.arange(n, device="cuda", dtype=torch.float32) / n  # the u of instance k times this
    all_q = q0[None].repeat(n, 1, 1, 1)
    all_q[:, 1] *= factor[:, None, None]
    start = all_q.clone()
    s = solver(g, torch.float32)
    s.set_bathymetry(bd)
    dt = s.cfl_dt(q0, 0.2)
    batch = Batch([g] * n, torch.float32)
    for k in range(n):
        batch.set_bathymetry(k, bd)
    batch.set_states(list(all_q))
    batch.step([dt] * n, 1)
    assert batch.check() == -1
    assert bool((all_q != start).flatten(1).any(1).all())  # every state was written
    for k in (0, 1, 16384, 65535, 65536, n - 1):
        one = start[k].clone()
        s.step(one, dt, 1)
        assert torch.equal(all_q[k], one), k
