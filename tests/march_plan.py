"""The rule by which a grid or an ensemble steps by strips (march kernel), as the
library's host code has it (march_plan, march_chunks), and its division into runs."""

MARCH_COLS = 56
MARCH_MIN_NODES = 1 << 20
MARCH_MIN_HEIGHT = 8
MARCH_LEAST_ROWS = 4


def cdiv(a, b):
    return -(-a // b)


def strips_of(nx):
    return cdiv(nx, MARCH_COLS)


def march_evals(strips, ny, chunks):
    return strips * (4 * ny + 12 * chunks)


def tile_evals(nx, ny):
    return 60 * cdiv(nx, 32) * cdiv(ny, 24)


def pays(march, tile, f64_walls=False):
    return 5 * march < 6 * tile if f64_walls else 4 * march < 5 * tile


def slots(dtype_bytes, cus):
    return cus * 4 * (2 if dtype_bytes == 8 else 3)


def run_rows(n, ny, walls):
    """First row of each of the n runs over ny rows, and ny."""
    rows = [0] + [ny * (5 * c - 1) // (5 * n - 2) if walls else ny * c // n for c in range(1, n)] + [ny]
    return rows


def least_rows(n, ny, walls):
    if n <= 1:
        return ny
    return 4 * ny // (5 * n - 2) if walls else ny // n


def plan(nx, ny, bc_x, bc_y, dtype_bytes, cus=256):
    """(runs of an inner strip, runs of a strip at a wall in x), or None: the grid steps by tiles.  Default step tile."""
    if cdiv(nx, 32) * cdiv(ny, 24) < 1024 or nx * ny < MARCH_MIN_NODES:
        return None
    s, most = strips_of(nx), max(1, ny // MARCH_MIN_HEIGHT)
    if bc_x and s < 3:
        return None
    k = slots(dtype_bytes, cus)
    chunks = max(1, min(2 * k // (2 * s + 1) if bc_x else k // s, most))
    if not pays(march_evals(s, ny, chunks), tile_evals(nx, ny), bc_x and bc_y and dtype_bytes == 8):
        return None
    wall = min(chunks + chunks // 4, most) if bc_x else 0
    if least_rows(max(chunks, wall), ny, bc_y) < MARCH_LEAST_ROWS:
        return None
    return chunks, wall


def batch_plan(grids, dtype_bytes, cus=256):
    """Runs per instance, or None.  grids: (nx, ny, bc_y)."""
    if sum(nx * ny for nx, ny, _ in grids) < MARCH_MIN_NODES:
        return None
    k = slots(dtype_bytes, cus)
    h = max(MARCH_MIN_HEIGHT, sum(strips_of(nx) * ny for nx, ny, _ in grids) // k)
    top = 2 * h
    while h < top and sum(strips_of(nx) * cdiv(ny, h) for nx, ny, _ in grids) > k:
        h += max(1, h // 32)
    chunks = [max(1, cdiv(ny, h)) for _, ny, _ in grids]
    if any(least_rows(n, ny, bc) < MARCH_LEAST_ROWS for n, (_, ny, bc) in zip(chunks, grids)):
        return None
    march = sum(march_evals(strips_of(nx), ny, n) for n, (nx, ny, _) in zip(chunks, grids))
    return chunks if pays(march, sum(tile_evals(nx, ny) for nx, ny, _ in grids)) else None
