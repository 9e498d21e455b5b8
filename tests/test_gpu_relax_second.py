"""Which way the second Newton iteration of the relaxation goes, and that both give it.

The host forms s(gam) and s'(gam) in extended precision from the state and its RK4
update, the series about gam = 1 and the bound under which the kernels take it.
The large steps pass that bound by so much that the series would miss the
iteration visibly: there the pass over the states has to have run."""

import numpy as np
import pytest

import oracle
from paper_2601_02540_amd import workloads as W
from gpu_util import STATE_FLOORS, dev, field_rel_err, host, solver

pytestmark = pytest.mark.gpu

LD = np.longdouble


def newton(g, q, b, dt):
    """The second iterate, the series' one, the series' bound over its limit, and the
    rounding of the second iterate: of the sums' terms in FP64, over the slope."""
    d = oracle.rk4(g, q, b, dt, 1).astype(LD) - q
    (h, u, v, w, eta), (dh, du, dv, dw, de) = q.astype(LD), d
    dx, dy = g.spacing()
    M = np.full(h.shape, dx * dy, LD)
    if g.bc_x == W.REFLECTING:
        M[:, [0, -1]] *= 0.5
    if g.bc_y == W.REFLECTING:
        M[[0, -1]] *= 0.5
    A, B, sq, sw = eta - h, de - dh, du * du + dv * dv, dw * dw
    lin, linw = 2 * (u * du + v * dv), 2 * w * dw

    def sums(gam):
        H = h + gam * dh
        Nl = h * (2 * A * B + gam * B * B) - dh * A * A
        parts = [0.5 * (dh * (u * u + v * v) + H * (lin + gam * sq)), (dh * w * w + H * (linw + gam * sw)) / 6,
                 0.5 * g.g * dh * (2 * h + 2 * b + gam * dh), g.lam / 6 * Nl / (h * H)]
        dlam = g.lam / 6 * (h * B * B * H - Nl * dh) / (h * H * H)
        ds = 0.5 * (dh * (lin + gam * sq) + H * sq) + (dh * (linw + gam * sw) + H * sw) / 6 + 0.5 * g.g * dh * dh + dlam
        return sum((M * p).sum() for p in parts), (M * ds).sum(), M * dlam, sum((M * abs(p)).sum() for p in parts)

    s0, s1, t1, size = sums(LD(1))
    gam1 = 1 - s0 / s1
    s, ds, _, _ = sums(gam1)
    second = gam1 - s / ds
    rho, delta = dh / (h + dh), gam1 - 1
    t = [t1]
    for _ in range(4):
        t.append(-rho * t[-1])
    c2, c3, c4 = (M * dh * (0.5 * sq + sw / 6)).sum() + t[1].sum(), t[2].sum(), t[3].sum()
    ser = delta ** 2 * (c2 + delta * (c3 + delta * c4))
    dser = s1 + delta * (2 * c2 + delta * (3 * c3 + 4 * delta * c4))
    x = 1 - abs(rho).max() * abs(delta)
    es, eds = abs(t[4]).sum() * abs(delta) ** 5 / x, 5 * abs(t[4]).sum() * delta ** 4 / x ** 2
    lim = LD(2) ** -56 * abs(dser)
    return second, gam1 - ser / dser, max(es / lim, eds * abs(ser) / (lim * abs(dser))), LD(2) ** -53 * size / abs(s1)


def start(bc, cfl):
    g = W.Grid(75, 52, -1.0, 1.5, -1.0, 1.0, bc, bc, 9.81, 500.0)
    q, b = W.random_state(g, 5, b_scale=0.1)
    q[1:4] *= 0.3
    q = oracle.init_aux(g, q, b)
    return g, q, b, oracle.cfl_dt(g, q, cfl)


@pytest.mark.parametrize("cfl", [0.3, 0.9])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.REFLECTING])
def test_small_steps_stay_within_the_bound(bc, cfl):
    """The steps of test_gpu_relax_series.py take the series, by a wide margin."""
    assert newton(*start(bc, cfl))[2] < 1e-2


@pytest.mark.parametrize("cfl", [2.6, 3.0])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.REFLECTING])
@pytest.mark.parametrize("path", ["fused", "pairs"])
def test_large_steps_take_the_pass(path, bc, cfl):
    """t_end = gam dt of one step.  Each node's terms of s take about 12 roundings, which
    the sums carry on (8 of them at the size of their parts, as the parts' errors
    are not all of one sign), and gam itself 4.  The increments are of the size of
    the state, so their own rounding is within that."""
    g, q, b, dt = start(bc, cfl)
    gam, series, over, rounding = newton(g, q, b, dt)
    tol = float(8 * rounding + 4 * 2.0 ** -53)
    assert 0.5 < gam < 1.5
    assert over > 1e3 and abs(series - gam) > 10 * tol, (over, series - gam, tol)
    s = solver(g)
    s.set_step_path(path)
    s.set_bathymetry(dev(b))
    qd = dev(q)
    t_end = s.step_relaxation(qd, dt, 1, 0.0)
    assert abs(t_end / dt - float(gam)) <= tol, (t_end / dt - float(gam), tol)
    ref = q + float(gam) * (oracle.rk4(g, q, b, dt, 1) - q)
    assert np.all(field_rel_err(host(qd), ref, STATE_FLOORS) <= 1e-12)
