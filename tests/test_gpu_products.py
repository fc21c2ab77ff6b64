"""The float64 products behind J^T J and the explicit Jacobian (k in padded slabs straight into LDS, 64- or
128-tiles, k in parts for few tiles) at the sizes where padding, clamped rows and parts can go wrong: element counts
that are no multiple of the slab (16), sample counts of one, either side of a slab and over several sample tiles,
one handle and enough handles for several tiles, against the oracle.  Bar 1e-10 of the largest entry, as
elsewhere for the float64 normal equations."""
import numpy as np
import pytest

import oracle as O
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.abs(a - b).max() / max(1e-300, np.abs(b).max())


@pytest.mark.parametrize("per_side,H,n,tile_rows", [(4, 1, 1, 0), (5, 2, 15, 0), (33, 3, 17, 0), (61, 11, 2085, 320),
                                                    (64, 34, 700, 0)])
def test_normal_equations_and_jacobian(per_side, H, n, tile_rows):
    S, eps = 4, 1e-2
    ctx = ctx_for(S, per_side=per_side, tile_rows=tile_rows)
    th, x, r = W.random_handles(H, H), W.random_points(n, n, 0.01, 0.99), W.random_vector(n, (n, 3))
    Ho, go = O.normal_equations(th, x, r, S, eps, per_side)
    JtJ, Jtr = ctx.jtj(dev(th), dev(x), dev(r), "fp64", "fp64")
    assert _rel(host(JtJ), Ho) < 1e-10 and _rel(host(Jtr), go) < 1e-10
    xj = x[:131]
    assert _rel(host(ctx.jacobian(dev(th), dev(xj))), O.jacobian(th, xj, S, eps, per_side)) < 1e-10
