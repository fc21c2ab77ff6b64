"""The mixed sweeps over grouped samples (cells of a square grid, the far field of a cell expanded from
its nodes) and over few samples (the tables split over blocks), against the FP64 path.

Sizes at the edges: one sample, wavefront and block remainders, either side of the smallest grouped call,
segment and element counts that leave partial 32-groups, cells without samples, all samples in one
cell, samples outside the outer boundary's box and not finite, handles longer than the cells, and near
factors that make most pairs near.

Tolerances: float32 pairs carry about 1e-6 of the largest colour (a few hundred terms of O(1) rounded at 2^-24
= 6e-8 and partly cancelling), the interpolated far field less than 1e-7; the bar is 1e-5 of the largest
colour (at least 1).  The gradients' bar is 1e-3 of the largest entry, as elsewhere for the mixed adjoint.
The float64 sweep over grouped samples is held to the direct one (itself held to the oracle) at 1e-12: sums of
some thousand O(1) terms round at 1e-13, the interpolation adds 1e-14.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)


def _straight(seed, H, length):
    rng = np.random.default_rng(np.random.SeedSequence(entropy=7000 + seed))
    a = rng.uniform(0.2, 0.8, size=(H, 2))
    ang = rng.uniform(0, 2 * np.pi, size=H)
    b = np.clip(a + length * np.stack([np.cos(ang), np.sin(ang)], 1), 0.02, 0.98)
    return np.ascontiguousarray(np.concatenate([a, b, W.draw_straight_colours(rng, H)], axis=1))


def _check(ctx, theta, x, rows=None):
    th, xd = dev(theta), dev(x)
    u = host(ctx.eval(th, xd, CBAR, "mixed"))
    r = host(ctx.eval(th, xd, CBAR, "fp64"))
    ok = np.isfinite(x).all(1) if rows is None else rows
    assert np.isfinite(r[ok]).all()
    assert np.abs(u[ok] - r[ok]).max(initial=0.0) < 1e-5 * max(1.0, np.abs(r[ok]).max(initial=0.0))
    g = W.random_vector(len(x), (len(x), 3)).astype(np.float32)
    g[~ok] = 0.0
    xg = np.where(ok[:, None], x, 0.5)
    a = host(ctx.vjp(th, dev(xg), dev(g), "mixed"))
    b = host(ctx.vjp(th, dev(xg), dev(g.astype(np.float64)), "fp64"))
    assert np.isfinite(b).all() and np.abs(a - b).max(initial=0.0) <= 1e-3 * np.abs(b).max(initial=0.0)
    return u


@pytest.mark.parametrize("n", [1, 63, 64, 65, 256, 257, 8191])
def test_few_samples(n):
    _check(ctx_for(8), W.random_handles(n, 5), W.random_points(n, n, 0.001, 0.999))


def test_few_segments_and_none():
    ctx = ctx_for(1)
    _check(ctx, W.random_handles(1, 1), W.random_points(1, 130, 0.01, 0.99))
    _check(ctx, np.zeros((0, 20)), W.random_points(2, 130, 0.01, 0.99))


@pytest.mark.parametrize("H,n", [(130, 8192), (131, 20011), (257, 100003)])
def test_grouped_samples(H, n):
    _check(ctx_for(31), W.random_handles(H, H), W.random_points(H, n, 1e-4, 1 - 1e-4))


def test_grouped_samples_empty_cells_strays_and_nan():
    ctx, th = ctx_for(32), W.random_handles(3, 128)
    x = W.random_points(3, 30000, 0.30, 0.34)                 # nearly all in one cell
    x[7] = (0.9, 0.1)
    _check(ctx, th, x)
    x = W.random_points(4, 30000, 0.001, 0.999)
    x[::1000] = 1.0 + W.random_points(5, 30, 0.01, 0.5)       # outside the boundary's box
    x[5::3000] = np.nan
    x[6] = (np.inf, 0.5)
    u = _check(ctx, th, x)
    assert np.isnan(u[5::3000]).all()


@pytest.mark.parametrize("length,nf", [(0.05, 1.0), (0.6, 1.0), (0.02, 20.0), (0.05, 0.5)])
def test_grouped_samples_long_handles_and_near_factors(length, nf):
    ctx = ctx_for(1, near_factor=nf, handle_model="straight")
    _check(ctx, _straight(1, 1501, length), W.random_points(6, 24001, 0.001, 0.999))


def test_grouped_samples_in_a_region():
    poly = np.array([[0.0, 0.0], [0.45, 0.0], [0.4, 1.0], [0.0, 1.0]])
    el = []
    for p, q, n in zip(poly, np.roll(poly, -1, 0), (57, 127, 50, 128)):
        t = np.linspace(0, 1, n + 1)[:, None]
        v = p * (1 - t) + q * t
        el.append(np.concatenate([v[:-1], v[1:]], 1))
    ctx = B.Context(segs_per_handle=16, elements=np.concatenate(el))
    x = W.random_points(8, 60000, 0.001, 0.999) * np.array([0.39, 1.0])
    th = W.random_handles(8, 90, spread=0.1, centre_lo=0.1, centre_hi=0.3)
    _check(ctx, th, x)
    ctx.close()


@pytest.mark.parametrize("H,S,n,width", [(256, 32, 400003, 0.37), (12, 8, 500000, 1.0)])
def test_levels_of_cells_in_a_narrow_region(H, S, n, width):
    """Enough samples for two and three levels of cells, in a region whose cells a side do not divide by the levels,
    half of the region without samples; few handles lie far from most cells, many fill them."""
    poly = np.array([[0.0, 0.0], [width, 0.0], [width, 1.0], [0.0, 1.0]])
    el = []
    for p, q, k in zip(poly, np.roll(poly, -1, 0), (57, 127, 57, 127)):
        t = np.linspace(0, 1, k + 1)[:, None]
        v = p * (1 - t) + q * t
        el.append(np.concatenate([v[:-1], v[1:]], 1))
    ctx = B.Context(segs_per_handle=S, elements=np.concatenate(el))
    x = W.random_points(n, n, 0.01, 0.99) * np.array([width, 1.0])
    x[: n // 2, 1] *= 0.3
    th = W.random_handles(H, H, spread=0.05, centre_lo=0.08, centre_hi=0.3)
    _check(ctx, th, x)
    u = host(ctx.eval(dev(th), dev(x), CBAR, "fp64"))
    r = host(ctx.eval(dev(th), dev(x[::101]), CBAR, "fp64"))               # few samples: the direct sums
    assert np.abs(u[::101] - r).max() < 1e-12 * max(1.0, np.abs(r).max())
    ctx.close()


def test_grouped_samples_view_off_16_bytes():
    ctx, th = ctx_for(32), dev(W.random_handles(9, 100))
    flat = dev(np.concatenate([[0.5], W.random_points(9, 20001, 0.01, 0.99).ravel()]))
    x = flat[1:].view(-1, 2)
    u = ctx.eval(th, x, CBAR, "mixed")
    assert torch.equal(u, ctx.eval(th, x.clone(), CBAR, "mixed")) or float((u - ctx.eval(th, x.clone(), CBAR, "mixed")).abs().max()) < 1e-6


@pytest.mark.parametrize("H,n", [(33, 20011), (64, 100003), (3, 262144)])
def test_grouped_samples_fp64(H, n):
    ctx, th = ctx_for(32), W.random_handles(H, H)
    x = W.random_points(H, n, 1e-4, 1 - 1e-4)
    x[::5000] = 1.0 + W.random_points(5, len(x[::5000]), 0.01, 0.5)       # outside the boundary's box
    x[3] = (np.nan, 0.5)
    u = host(ctx.eval(dev(th), dev(x), CBAR, "fp64"))
    idx = np.r_[0:3, 4:2000, n - 3000:n]
    r = host(ctx.eval(dev(th), dev(x[idx]), CBAR, "fp64"))                 # few samples: the direct sums
    assert np.isnan(u[3]).all() and np.isfinite(np.delete(u, 3, 0)).all()
    assert np.abs(u[idx] - r).max() < 1e-12 * max(1.0, np.abs(r).max())


@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 1025])
def test_few_samples_fp64_matches_oracle(n):
    th, x, g = W.random_handles(n, 9), W.random_points(n, n, 0.01, 0.99), W.random_vector(n, (n, 3))
    ctx = ctx_for(8)
    u, uo = host(ctx.eval(dev(th), dev(x), CBAR, "fp64")), O.evaluate(th, x, CBAR, 8, 1e-2)
    assert np.abs(u - uo).max() < 1e-10
    a, b = host(ctx.vjp(dev(th), dev(x), dev(g), "fp64")), O.vjp(th, x, g, 8, 1e-2)
    assert np.abs(a - b).max() < 1e-10 * np.abs(b).max()


# 340,000 samples: four wavefronts to a unit of 64 samples; 400,000: one.  130 segments and the elements leave every
# fourth-bit share uneven, and samples on the segments fill the lists.
@pytest.mark.parametrize("n", [340000, 400000])
def test_units_of_four_wavefronts_and_of_one(n):
    ctx, theta = ctx_for(1, handle_model="straight"), _straight(21, 130, 0.05)
    x = W.random_points(22, n, 1e-3, 1 - 1e-3)
    t = np.arange(2000) / 2000.0
    x[:2000] = theta[7, 0:2] + t[:, None] * (theta[7, 2:4] - theta[7, 0:2]) + 1e-5
    u, r = (host(ctx.eval(dev(theta), dev(x), CBAR, p)) for p in ("mixed", "fp64"))
    assert np.isfinite(r).all()
    assert np.abs(u - r).max() < 1e-5 * max(1.0, np.abs(r).max())
