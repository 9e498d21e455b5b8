"""Misfits of a kept rollout with more rows than the recording launch has blocks."""

import numpy as np
import pytest
import torch

from paper_2601_02540_amd import workloads as W
from gpu_util import dev, host, solver

pytestmark = pytest.mark.gpu

ROW_BLOCKS = 4096  # MAX_RECORD_BLOCKS of sgn_adjoint.hip


@pytest.mark.parametrize("steps", [ROW_BLOCKS, ROW_BLOCKS + 1, 2 * ROW_BLOCKS + 300])
def test_loss_of_many_rows(steps):
    g = W.Grid(4, 5, 0.0, 0.4, 0.0, 0.5, W.PERIODIC, W.REFLECTING, 9.81, 500.0)
    rng = np.random.default_rng(2)
    b = 0.05 * rng.standard_normal((5, 4))
    zeta0 = 1.0 + 0.01 * rng.standard_normal((5, 4))
    nodes = dev(np.array([3, 17, 8]))
    target = dev(1.0 + 0.01 * rng.standard_normal((steps, 3)))
    s = solver(g)
    s.set_bathymetry(dev(b))
    dt = 1e-3
    results = []
    for store in ((4 * steps + 1) * 5 * 20 * 8, 0):  # every step kept: one launch for all rows; segments of about sqrt(steps)
        s.set_adjoint_store(store)
        results.append(s.gauge_loss_grad(dev(zeta0), steps, dt, nodes, target))
    series = s.gauge_series(dev(zeta0), steps, dt, nodes)
    loss = float((0.5 * (series - target) ** 2).sum())
    assert abs(results[0][0] - loss) <= 1e-12 * loss  # sums of up to 25000 terms in another order
    assert results[0][0] == results[1][0]
    assert np.array_equal(host(results[0][1]), host(results[1][1]))
    assert np.array_equal(host(results[0][2]), host(results[1][2]))
    assert torch.isfinite(series).all()
