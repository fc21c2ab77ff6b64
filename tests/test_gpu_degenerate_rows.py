"""Handles of no length in the mixed normal equations: no integral and no derivative, so rows of zeros in J^T J (over
tiles of samples and over cells) and parameters that a step leaves as they are, exactly."""
import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)
GONE = (3, 17)


def _theta(model, H):
    if model == "cubic":
        th = W.random_handles(5, H, spread=0.03)
        th[list(GONE), :8] = np.tile(th[list(GONE), :2], 4)
        return th
    rng = np.random.default_rng(6)
    a = rng.uniform(0.2, 0.8, (H, 2))
    th = np.concatenate([a, a + 0.03, W.draw_straight_colours(rng, H)], 1)
    th[list(GONE), 2:4] = th[list(GONE), :2]
    return th


@pytest.mark.parametrize("model,S", [("straight", 1), ("straight", 3), ("cubic", 1), ("cubic", 8)])
@pytest.mark.parametrize("gram", ["bf16x3_mfma", "fp32_mfma"])
def test_rows_of_zeros(model, S, gram):
    ctx, th = ctx_for(S, handle_model=model), _theta(model, 24)
    x = W.random_points(7, 5000, 1e-3, 1 - 1e-3)
    J, g = ctx.jtj(dev(th), dev(x), dev(W.random_vector(8, (len(x), 3)), torch.float32), gram, "mixed")
    J, g = host(J).reshape(24, th.shape[1], -1), host(g).reshape(24, -1)
    assert not J[list(GONE)].any() and not g[list(GONE)].any()
    assert (np.abs(J).max((1, 2)) > 0).sum() == 22


@pytest.mark.parametrize("model,S", [("straight", 1), ("cubic", 8)])
@pytest.mark.parametrize("tile_rows", [0, 4096])                    # over cells, over tiles
def test_step_leaves_them(model, S, tile_rows):
    ctx, th = ctx_for(S, handle_model=model, tile_rows=tile_rows), _theta(model, 40)
    xd = dev(W.random_points(9, 60000, 1e-3, 1 - 1e-3))
    T = ctx.eval(dev(th), xd, CBAR, "fp64") + 0.05 * dev(W.random_vector(10, (len(xd), 3)))
    t, st = dev(th), B.new_lm_state(1.0)
    ctx.profile(True)
    ctx.lm_step(t, xd, T, st, "bf16x3_mfma", "mixed")
    tiles = ctx.profile_read()["beta_rows"][1] > 0
    ctx.profile(False)
    assert st.accepted and tiles == (tile_rows > 0)
    moved = np.abs(host(t) - th).max(1)
    assert not moved[list(GONE)].any() and (moved > 0).sum() == 38


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n", [500, 60000])                         # direct and grouped sums
@pytest.mark.parametrize("what", ["jump", "all"])
def test_values_that_are_not_finite_show(value, n, what):
    """A handle of no length (or of none that is a number) hides no jump that is not finite."""
    th = _theta("straight", 400)
    th[GONE[0], 5 if what == "jump" else slice(None)] = value
    u = ctx_for(1, handle_model="straight").eval(dev(th), dev(W.random_points(11, n, 1e-3, 1 - 1e-3)), CBAR, "mixed")
    assert not np.isfinite(host(u)).all(1).any()
