"""The mixed LM step with its normal equations over grid cells (split-BF16 Gram) against the FP64 step and
against the same step over tiles of samples (a context with a tile size of its own).

Sizes at the edges: cells with some 100 samples (fewer than nodes, and samples in part of a cell, are in
test_gpu_cell_normal_regions.py), samples nearly all in a few cells, cells without samples, samples outside the outer boundary's box, segment counts that leave
partial 32-groups of the near bitmaps, one segment and many segments a handle, every handle near (no cell is
worth it: tiles), and near factors either side of the quadrature's reach.

Tolerance: helpers.mixed_step_tol, the condition of the damped normal equations times float32 rounding, as
for the steps over tiles.
"""
import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host, log, mixed_step_tol

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)
LAM = 1.0


def _straight(seed, H, length):
    rng = np.random.default_rng(np.random.SeedSequence(entropy=8000 + seed))
    a = rng.uniform(0.2, 0.8, size=(H, 2))
    ang = rng.uniform(0, 2 * np.pi, size=H)
    b = np.clip(a + length * np.stack([np.cos(ang), np.sin(ang)], 1), 0.02, 0.98)
    return np.ascontiguousarray(np.concatenate([a, b, W.draw_straight_colours(rng, H)], axis=1))


def _step(ctx, th0, x, T, gram, prec):
    th, st = th0.clone(), B.new_lm_state(LAM, 0)
    ctx.lm_step(th, x, T, st, gram, prec)
    return host(th - th0).ravel(), st


def _check(theta, x, S, model, nf=1.0):
    ctx, tiles = ctx_for(S, near_factor=nf, handle_model=model), ctx_for(S, near_factor=nf, handle_model=model, tile_rows=4096)
    th0, xd = dev(theta), dev(x)
    T = ctx.eval(th0, xd, CBAR, "fp64") + 0.05 * dev(W.random_vector(71, (len(x), 3)))
    d64, s64 = _step(ctx, th0, xd, T, "fp64", "fp64")
    dc, sc = _step(ctx, th0, xd, T, "bf16x3_mfma", "mixed")
    dt, st = _step(tiles, th0, xd, T, "bf16x3_mfma", "mixed")
    assert s64.accepted == sc.accepted == st.accepted == 1
    JtJ, _ = ctx.jtj(th0, xd, torch.zeros_like(T), "fp64", "fp64")
    tol = mixed_step_tol(host(JtJ), LAM)
    ec, et = (np.abs(d - d64).max() / np.abs(d64).max() for d in (dc, dt))
    log(f"{model} S={S} H={len(theta)} N={len(x)}: cells {ec:.2e}, tiles {et:.2e}, bar {tol:.2e}")
    assert ec < tol and et < tol
    assert abs(sc.loss_after - s64.loss_after) < 1e-5 * s64.loss_after


@pytest.mark.parametrize("S,H,n", [(32, 60, 65536), (31, 33, 20011), (1, 40, 30001)])
def test_cubic_handles(S, H, n):
    _check(W.random_handles(H, H, spread=0.03), W.random_points(H, n, 1e-3, 1 - 1e-3), S, "cubic")


@pytest.mark.parametrize("S,length,nf", [(1, 0.02, 1.0), (1, 0.02, 3.0), (4, 0.05, 1.0)])
def test_straight_handles(S, length, nf):
    _check(_straight(S, 301, length), W.random_points(9, 50021, 1e-3, 1 - 1e-3), S, "straight", nf)


def test_tiles_where_cells_do_not_serve():
    x = W.random_points(10, 30000, 1e-3, 1 - 1e-3)
    _check(_straight(2, 101, 0.7), x, 1, "straight")
    _check(_straight(3, 101, 0.02), x, 1, "straight", nf=0.5)


def test_strays_and_clustered_samples():
    th = W.random_handles(5, 40, spread=0.03)
    x = W.random_points(11, 60000, 1e-3, 1 - 1e-3)
    x[::500] = 1.0 + W.random_points(12, len(x[::500]), 0.01, 0.5)
    _check(th, x, 16, "cubic")
    x = 0.4 + 0.2 * W.random_points(13, 60000, 1e-3, 1 - 1e-3)
    x[::3] = W.random_points(14, len(x[::3]), 1e-3, 1 - 1e-3)
    _check(th, x, 16, "cubic")


# from 204,800 samples on the far rows of items of 16 segments take two levels of cells: the smallest grid (20 cells a
# side), an odd one (21, made even), a last item of one straight handle, and samples that leave cells of 2 x 2 empty or
# in part empty
@pytest.mark.parametrize("S,H,n,model,part", [(16, 12, 204801, "cubic", 0), (32, 9, 250007, "cubic", 0),
                                              (8, 41, 215000, "straight", 0), (16, 12, 230000, "cubic", 1)])
def test_far_rows_over_two_levels(S, H, n, model, part):
    th = W.random_handles(H, H, spread=0.1) if model == "cubic" else _straight(H, H, 0.1)
    x = W.random_points(H + n, n, 1e-3, 1 - 1e-3)
    if part:
        x[:] = np.where(np.arange(n)[:, None] % 3 == 0, x, 0.42 + 0.16 * x)
        x[x[:, 0] < 0.23] += 0.5
        x = np.minimum(x, 1 - 1e-3)
    _check(th, x, S, model)
