"""Grouped float64 samples in domains far from the origin: segments and elements are far from a cell by their true
distance, wherever the domain lies.

All coordinates are multiples of 2^-20, so that a shift by whole numbers up to 1e7 is exact.  Nodes and samples are placed
from the grid's origin, so that the bar is that of the unit square (test_gpu_cells.py): 1e-12.
"""
import numpy as np
import pytest

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import dev, host

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)


def _grid(a):
    return np.round(np.asarray(a) * 2.0 ** 20) / 2.0 ** 20


def _square(n=128):
    c = np.array([(0.0, 0.0), (1.0, 0.0), (1.0, 1.0), (0.0, 1.0), (0.0, 0.0)])
    v = np.concatenate([c[i] + (np.arange(n) / n)[:, None] * (c[i + 1] - c[i]) for i in range(4)] + [c[:1]])
    return np.concatenate([v[:-1], v[1:]], 1)


@pytest.mark.parametrize("shift", [(0.0, 0.0), (1e6, -2e6), (1e7, 3e6), (-1e7, 1e7)])
def test_shifted_domain_fp64(shift):
    rng = np.random.default_rng(11)
    a = rng.uniform(0.1, 0.9, (400, 2))
    ang = rng.uniform(0, 2 * np.pi, 400)
    th = np.concatenate([_grid(a), _grid(a + 0.04 * np.stack([np.cos(ang), np.sin(ang)], 1)), W.draw_straight_colours(rng, 400)], 1)
    x = _grid(W.random_points(12, 60000, 1e-3, 1 - 1e-3))
    at = np.array(shift)
    ctx = B.Context(segs_per_handle=1, elements=_square() + np.tile(at, 2), handle_model="straight")
    t = dev(np.concatenate([th[:, :2] + at, th[:, 2:4] + at, th[:, 4:]], 1))
    u, r = (host(ctx.eval(t, dev(y + at), CBAR, "fp64")) for y in (x, x[::31]))
    ctx.close()
    bar = 1e-12 * max(1.0, np.abs(r).max())
    print(f"{shift}: {np.abs(u[::31] - r).max():.1e}, bar {bar:.1e}")
    assert np.abs(u[::31] - r).max() < bar
