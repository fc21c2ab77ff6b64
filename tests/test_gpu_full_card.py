"""Calls on a card whose memory is taken but for some tens of MiB: where the grouped sums' workspaces find no memory, the
calls take their other form, with the same result.

Every kernel that may run has run before, in other contexts, so that the card is full only for the library's own
allocations.
"""
import contextlib

import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import dev, host, mixed_step_tol

pytestmark = pytest.mark.gpu
CBAR = (0.3, 0.5, 0.7)
MIB = 1 << 20


@contextlib.contextmanager
def _full(leave):
    """All of the card's memory taken but `leave` bytes and what is no multiple of 2 MiB."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    spare = torch.empty(leave, dtype=torch.uint8, device="cuda")
    held, size = [], 1 << 36
    try:
        while size >= 2 * MIB:
            try:
                held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
            except torch.OutOfMemoryError:
                size //= 2
        del spare
        torch.cuda.empty_cache()
        yield
    finally:
        torch.cuda.synchronize()
        held.clear()
        torch.cuda.empty_cache()


def _scene(H, n):
    rng = np.random.default_rng(H)
    a = rng.uniform(0.2, 0.8, (H, 2))
    th = np.concatenate([a, a + 0.02, W.draw_straight_colours(rng, H)], 1)
    x = torch.rand(n, 2, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(H)) * 0.998 + 1e-3
    return dev(th), x


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-5)])
def test_eval(prec, bar):
    th, x = _scene(64, 6_000_000)                # 24 bytes a sample: 144 MB of cell order
    kw = dict(segs_per_handle=1, elems_per_side=32, handle_model="straight")
    want, few = B.Context(**kw), x[:9000].contiguous()
    r, rf = want.eval(th, x, CBAR, prec), want.eval(th, few, CBAR, prec)
    ctx, out = B.Context(**kw), torch.empty_like(r)
    ctx.eval(th, few, CBAR, prec, out=out[:9000])
    with _full(64 * MIB):
        ctx.eval(th, x, CBAR, prec, out=out)
        torch.cuda.synchronize()
    big = max(1.0, float(r.abs().max()))
    assert float((out - r).abs().max()) < bar * big and float((out[:9000] - rf).abs().max()) < bar * big
    ctx.close(), want.close()


def test_lm_step():
    """A context that has the workspaces of the tiles (bem_jtj in split BF16, a step of another Gram) but not of the cells."""
    th, x = _scene(60, 2_000_000)                # 35 cells a side, 57 KiB each
    kw = dict(segs_per_handle=1, elems_per_side=32, handle_model="straight")
    want, ctx = B.Context(**kw), B.Context(**kw)
    T = want.eval(th, x, CBAR, "fp64") + 0.05 * torch.randn(len(x), 3, dtype=torch.float64, device="cuda",
                                                            generator=torch.Generator("cuda").manual_seed(1))
    r32 = torch.zeros(len(x), 3, device="cuda")

    def step(c, gram, prec):
        t, st = th.clone(), B.new_lm_state(1.0)
        c.lm_step(t, x, T, st, gram, prec)
        return t, st

    t64, s64 = step(want, "fp64", "fp64")
    JtJ, _ = want.jtj(th, x, torch.zeros_like(T), "fp64", "fp64")
    want.profile(True)
    step(want, "bf16x3_mfma", "mixed")                       # the cells' kernels
    assert want.profile_read()["beta_rows"][1] == 0
    want.close()
    ctx.jtj(th, x, r32, "bf16x3_mfma", "mixed")
    step(ctx, "fp32_mfma", "mixed")
    ctx.profile(True)
    t, st = th.clone(), B.new_lm_state(1.0)
    with _full(32 * MIB):
        ctx.lm_step(t, x, T, st, "bf16x3_mfma", "mixed")
        tiles = ctx.profile_read()["beta_rows"][1]
    d, d64 = host(t - th), host(t64 - th)
    assert tiles > 0 and st.accepted == s64.accepted == 1
    assert np.abs(d - d64).max() < mixed_step_tol(host(JtJ), 1.0) * np.abs(d64).max()
    ctx.close()


def test_jtj_fp64():
    """32,768 samples in tiles of 16,384 where a tile of all of them (298 MB) does not fit."""
    th, x = dev(W.random_handles(4, 4, spread=0.1)), dev(W.random_points(5, 32768, 0.01, 0.99))
    r = dev(W.random_vector(6, (len(x), 3)))
    want, ctx = B.Context(segs_per_handle=4), B.Context(segs_per_handle=4)
    J, g = want.jtj(th, x, r)
    want.close()
    few = x[:2000].contiguous()
    ctx.jtj(th, few, r[:2000].contiguous())                  # all but the tile of samples
    ctx.vjp(th, x, r)
    with _full(160 * MIB):
        J1, g1 = ctx.jtj(th, x, r)
        torch.cuda.synchronize()
    assert float((J1 - J).abs().max()) < 1e-12 * float(J.abs().max())
    assert float((g1 - g).abs().max()) < 1e-12 * float(g.abs().max())
    ctx.close()
