"""sgn_profile_stages on a small grid times the launches that sgn_step makes there."""

import pytest
import torch

import oracle
from paper_2601_02540_amd import workloads as W
from gpu_util import dev, solver

pytestmark = pytest.mark.gpu


def problem():
    p = W.gaussian_bump_periodic(64, seed=1)
    return p.grid, oracle.init_aux(p.grid, p.q0, p.b), p.b


def profiled(steps, tile=None):
    g, q, b = problem()
    s = solver(g)
    if tile:
        s.set_tile_y(tile)
    s.set_bathymetry(dev(b))
    qd = dev(q)
    dt = s.cfl_dt(qd, 0.2)
    return s.profile_stages(qd, dt, steps), qd, dt


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 6, 8, 10])
def test_state_and_form(steps):
    ms, qd, dt = profiled(steps)
    assert ms[0] > 0.0 and ms[1:] == [0.0, 0.0, 0.0]
    g, q, b = problem()
    s = solver(g)
    s.set_bathymetry(dev(b))
    ref = dev(q)
    s.step(ref, dt, steps + steps % 2)
    assert torch.equal(qd, ref)


def test_times_the_two_step_launches():
    """Two steps a launch take clearly less than the tile kernel's one step a launch, twice."""
    small = sorted(profiled(200)[0][0] for _ in range(5))[2]
    tile = sorted(profiled(200, 16)[0][0] for _ in range(5))[2]
    assert small < 0.85 * tile, (small, tile)
