"""The FP64 gauge gradient where its sums cancel: gauges in resting and in moving water.

grad_b = bbar - grad_zeta0, two sums of the size of the misfits.  Where the water
rests the surface does not depend on the bottom, so they cancel, and the digits
that are left are the rounding of every evaluation before.  Such a gradient is
compared with the oracle relative to what cancels, and with the bits on record."""

import os

import numpy as np
import pytest
import torch

import oracle
from paper_2601_02540_amd import workloads as W
from gpu_util import dev, host, solver

pytestmark = pytest.mark.gpu

RECORD = os.path.join(os.path.dirname(__file__), "golden", "gauge_gradient_at_rest.txt")
BCS = {"pp": (0, 0), "ww": (1, 1), "pw": (0, 1), "wp": (1, 0)}
NX, NY, STEPS, DT = 75, 52, 9, 1.5e-3
SAMPLE = 61  # every so many nodes of grad_b are on record


def case(bc):
    """A bump of bounded extent, water at rest elsewhere; +, -, * and / only, so the inputs are the same everywhere."""
    g = W.Grid(NX, NY, 0.0, 0.1 * NX, 0.0, 0.1 * NY, *BCS[bc], 9.81, 500.0)
    x, y = np.arange(NX)[None, :] / NX, np.arange(NY)[:, None] / NY
    b = 0.8 * x * (1.0 - x) * (y - 0.3) * (1.0 - y)
    r2 = 16.0 * ((x - 0.3) * (x - 0.3) + (y - 0.5) * (y - 0.5))
    zeta0 = 1.0 + 0.1 * np.maximum(0.0, 1.0 - r2) * np.maximum(0.0, 1.0 - r2)
    nodes = np.array([26 * NX + 22, 20 * NX + 35, 30 * NX + 60, 8 * NX + 66, 45 * NX + 58, 3 * NX + 71])
    n, k = np.arange(STEPS)[:, None], np.arange(len(nodes))[None, :]
    target = 1.0 + 0.01 * ((7 * n + 5 * k) % 11) / 11.0
    return g, zeta0, b, nodes, target


def gradient(bc, path="fused"):
    g, zeta0, b, nodes, target = case(bc)
    s = solver(g)
    s.set_step_path(path)
    s.set_bathymetry(dev(b))
    return s.gauge_loss_grad(dev(zeta0), STEPS, DT, dev(nodes), dev(target))


def read_record():
    rec = {}
    with open(RECORD) as f:
        for line in f:
            if not line.startswith("#"):
                name, *values = line.split()
                rec[name] = [float.fromhex(v) for v in values]
    return rec


@pytest.mark.parametrize("bc", sorted(BCS))
def test_gradient_on_record(bc):
    """Loss and grad_b to the bit."""
    loss, _, gb = gradient(bc)
    rec = read_record()[bc]
    assert loss == rec[0]
    assert host(gb).reshape(-1)[::SAMPLE].tolist() == rec[1:]


@pytest.mark.parametrize("path", ["fused", "pairs"])
@pytest.mark.parametrize("bc", sorted(BCS))
def test_gradient_relative_to_what_cancels(bc, path):
    """Against the oracle: each of the 4 evaluations of the 9 steps and of their
    reverse adds about 40 roundings of what its sums hold, which is what the seeds
    brought, at most the largest of |grad_zeta0|: 2 * 9 * 4 * 40 * 2^-53 = 3.2e-13."""
    g, zeta0, b, nodes, target = case(bc)
    loss_ref, gz_ref, gb_ref = oracle.gauge_loss_grad(g, zeta0, b, DT, STEPS, nodes, target)
    loss, gz, gb = gradient(bc, path)
    size = np.abs(gz_ref).max()
    rest = np.s_[:, 50:70]  # around the gauges that the bump has not reached
    assert np.abs(gb_ref[rest]).max() <= 1e-6 * np.abs(gz_ref[rest]).max()
    assert abs(loss - loss_ref) <= 1e-13 * loss_ref
    assert np.abs(host(gz) - gz_ref).max() <= 3.2e-13 * size
    assert np.abs(host(gb) - gb_ref).max() <= 3.2e-13 * size
