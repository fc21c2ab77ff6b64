"""Colours at samples on end points: of handles without regularisation, in mixed precision (a near pair's float32 form is
not finite there and has to leave no trace), and of outer elements to the smallest distances that float64 holds."""
import numpy as np
import pytest
import torch

from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)


@pytest.mark.parametrize("H,n", [(40, 300), (900, 30000)])          # direct, grouped
@pytest.mark.parametrize("nf", [0.5, 1.0])
def test_on_handle_ends(H, n, nf):
    rng = np.random.default_rng(H)
    a = rng.uniform(0.15, 0.85, (H, 2))
    b = a + rng.choice([0.2, 0.05, 0.005], H)[:, None] * rng.uniform(-0.7, 0.7, (H, 2))
    th = dev(np.concatenate([a, b, W.draw_straight_colours(rng, H)], 1))
    x = rng.uniform(0.01, 0.99, (n, 2))
    x[:80] = np.concatenate([a[:40], b[:40]])
    ctx = ctx_for(1, eps=0.0, near_factor=nf, per_side=32, handle_model="straight")
    u, r = (host(ctx.eval(th, dev(x), CBAR, p)) for p in ("mixed", "fp64"))
    assert np.isfinite(r).all() and np.isfinite(u).all()
    assert np.abs(u - r).max() < 1e-4 * max(1.0, np.abs(r).max())


@pytest.mark.parametrize("n", [300, 30000])
@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-5)])
def test_beside_element_ends(n, prec, bar):
    """Angles do not change with the distance to the corner on a line into it.  Where the terms of an angle are denormal
    (within 1e-306 of the corner) it may be off by pi / 16, 1/32 of a turn: of the boundary value, at two elements.  (Below
    1e-320 the terms have no digits left.)"""
    ctx, th = ctx_for(4, per_side=32), dev(W.random_handles(3, 300))
    x = np.random.default_rng(1).uniform(0.01, 0.99, (n, 2))
    d = np.array([1e-290, 1e-300, 3e-304, 1e-308, 1e-310, 1e-315, 1e-320])
    x[:7], x[7:14] = d[:, None] * [1.0, 1.0], d[:, None] * [2.0, 1.0]
    u = host(ctx.eval(th, dev(x), CBAR, prec))
    assert np.isfinite(u).all()
    big = max(1.0, np.abs(host(ctx.boundary_solve(th)[1])).max(), np.abs(u).max())
    for i in (0, 7):
        assert np.abs(u[i:i + 3] - u[i]).max() < bar * big
        assert np.abs(u[i + 3:i + 7] - u[i]).max() < (2 / 32 + bar) * big


def test_gradients_beside_element_ends():
    """One such sample among others leaves the others' gradients finite."""
    ctx, th = ctx_for(4, per_side=32), dev(W.random_handles(3, 30))
    x = W.random_points(4, 300, 0.01, 0.99)
    x[:3] = [[1e-310, 1e-310], [1.0, 1e-315], [1e-309, 0.0]]
    g = W.random_vector(5, (300, 3))
    for prec, dt in (("fp64", torch.float64), ("mixed", torch.float32)):
        assert bool(torch.isfinite(ctx.vjp(th, dev(x), dev(g, dt), prec)).all())
        assert bool(torch.isfinite(ctx.jtj(th, dev(x), dev(g, dt), "fp64", prec)[0]).all())
