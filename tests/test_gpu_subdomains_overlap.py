"""Subdomains' steps side by side: the same steps as one after the other, on the caller's stream and ordered with it;
an error of one undoes those after it; subdomains that share a context are taken in turn.

Steps are compared with those of contexts of their own on the same samples: the same kernels on the same inputs, but
for the order of float64 atomics, so 1e-12 of theta in float64.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import dev, host

pytestmark = pytest.mark.gpu
POLY = [[(i / 5, 0.0), ((i + 1) / 5, 0.0), ((i + 1) / 5, 1.0), (i / 5, 1.0)] for i in range(5)]


def _elements(poly, n=24):
    out = []
    for p, q in zip(poly, poly[1:] + poly[:1]):
        v = np.array(p) + (np.arange(n + 1) / n)[:, None] * (np.array(q) - np.array(p))
        out.append(np.concatenate([v[:-1], v[1:]], 1))
    return np.concatenate(out)


def _scene(D, n, seed):
    rng = np.random.default_rng(seed)
    ctxs = [B.Context(elements=_elements(POLY[d]), segs_per_handle=1, eps=1e-2, handle_model="straight") for d in range(D)]
    ths = []
    for d in range(D):
        a = np.stack([rng.uniform(d / 5 + 0.03, d / 5 + 0.15, 12 + d), rng.uniform(0.1, 0.8, 12 + d)], 1)
        ths.append(dev(np.concatenate([a, a + [0.02, 0.06], 0.5 * W.draw_straight_colours(rng, 12 + d)], axis=1)))
    x = W.random_points(seed, n, 1e-3, 1 - 1e-3)
    labels = np.minimum((x[:, 0] * 5).astype(np.int32), D - 1)
    return ctxs, ths, dev(x), dev(W.random_vector(seed + 1, (n, 3))), torch.from_numpy(labels).cuda()


def _in_turn(ths, x, T, labels, D):
    out = []
    for d in range(D):
        ctx = B.Context(elements=_elements(POLY[d]), segs_per_handle=1, eps=1e-2, handle_model="straight")
        m = labels == d
        th, st = ths[d].clone(), B.new_lm_state(1.0, compat=1)
        st.data_count = len(x)
        ctx.lm_step(th, x[m].contiguous(), T[m].contiguous(), st, "fp64", "fp64")
        out.append((host(th), st.accepted, st.loss_after))
    return out


@pytest.mark.parametrize("D,n", [(2, 3000), (5, 9001)])          # fewer subdomains than threads, and more
def test_side_by_side(D, n):
    ctxs, ths, x, T, labels = _scene(D, n, 40 + D)
    want = _in_turn(ths, x, T, labels, D)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                                 # inputs written on the caller's stream just before
        late = [torch.zeros_like(t) for t in ths]
        torch.cuda._sleep(2_000_000)
        for a, b in zip(late, ths):
            a.copy_(b)
        states = [B.new_lm_state(1.0, compat=1) for _ in range(D)]
        B.lm_step_subdomains(ctxs, late, x, T, labels, states, "fp64", "fp64")
        got = [(t + 0.0).cpu().numpy() for t in late]
    for g, st, (w, acc, loss) in zip(got, states, want):
        assert st.accepted == acc
        assert np.abs(g - w).max() <= 1e-12 * np.abs(w).max()
        assert abs(st.loss_after - loss) <= 1e-12 * loss


def test_error_undoes_the_steps_after_it():
    ctxs, ths, x, T, labels = _scene(3, 4000, 50)
    T[labels == 1] = float("nan")                                 # subdomain 1 is refused: no finite loss
    want = _in_turn(ths, x, T, labels, 1)
    keep = [t.clone() for t in ths]
    states = [B.new_lm_state(1.0, compat=1) for _ in range(3)]
    blank = bytes(B.new_lm_state(1.0, compat=1))
    with pytest.raises(B.BemError):
        B.lm_step_subdomains(ctxs, ths, x, T, labels, states, "fp64", "fp64")
    assert np.abs(host(ths[0]) - want[0][0]).max() <= 1e-12 * np.abs(want[0][0]).max()
    assert torch.equal(ths[2], keep[2]) and bytes(states[2]) == blank
    assert ctypes.sizeof(states[2]) == len(blank)


def test_shared_context_in_turn():
    ctxs, ths, x, T, labels = _scene(2, 3000, 60)
    a, b = [t.clone() for t in ths], [t.clone() for t in ths]
    sa, sb = ([B.new_lm_state(1.0) for _ in range(2)] for _ in range(2))
    B.lm_step_subdomains([ctxs[0], ctxs[0]], a, x, T, labels, sa, "fp64", "fp64")
    for d in range(2):
        m = labels == d
        sb[d].data_count = len(x)
        ctxs[0].lm_step(b[d], x[m].contiguous(), T[m].contiguous(), sb[d], "fp64", "fp64")
    for p, q in zip(a, b):
        assert np.abs(host(p) - host(q)).max() <= 1e-12 * np.abs(host(q)).max()
