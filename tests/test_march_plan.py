"""Runs of rows of the march kernel's plans: how short they get, and that none is lost."""

import random

from march_plan import MARCH_LEAST_ROWS, MARCH_MIN_HEIGHT, batch_plan, cdiv, least_rows, plan, run_rows


def test_runs_of_single_grids():
    rng = random.Random(3)
    taken = 0
    for _ in range(4000):
        nx, ny = int(2 ** rng.uniform(2, 15)), int(2 ** rng.uniform(2, 15))
        bc_x, bc_y, size = rng.randint(0, 1), rng.randint(0, 1), rng.choice((4, 8))
        p = plan(nx, ny, bc_x, bc_y, size)
        if p is None:
            continue
        taken += 1
        for n in filter(None, p):
            rows = run_rows(n, ny, bc_y)
            least = min(b - a for a, b in zip(rows, rows[1:]))
            assert rows[0] == 0 and rows[-1] == ny
            assert least == least_rows(n, ny, bc_y) >= MARCH_LEAST_ROWS, (nx, ny, n)
            assert n == 1 or least >= (4 * MARCH_MIN_HEIGHT // 5 if bc_y else MARCH_MIN_HEIGHT)
    assert taken > 300


def test_runs_of_instances():
    """Every height an instance can have against every run height of the rule."""
    for h in (8, 9, 12, 27, 100):
        for ny in range(4, 700):
            n = cdiv(ny, h)
            for walls in (0, 1):
                rows = run_rows(n, ny, walls)
                assert min(b - a for a, b in zip(rows, rows[1:])) == least_rows(n, ny, walls) >= MARCH_LEAST_ROWS


def test_grids_that_step_faster_on_tiles():
    """FP64 with walls on both axes: short runs, or a last strip of one column, step on tiles."""
    for nx, ny in ((1065, 1000), (300, 3600), (1024, 1024)):
        assert plan(nx, ny, 1, 1, 8) is None
    for nx, ny, bc, size in ((1065, 1000, 0, 8), (1200, 900, 1, 8), (1448, 1448, 1, 8), (1500, 900, 1, 4)):
        assert plan(nx, ny, bc, bc, size) is not None


def test_small_instances_make_a_plan():
    assert batch_plan([(4, 4, 1)] * 65600, 4) is not None
    assert batch_plan([(120, 9, 1)] * 1000, 8) is not None
