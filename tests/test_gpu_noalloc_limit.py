"""bem_vjp_noalloc up to the last sizes that its 64 MiB hold with the fewest chunks of samples (its finer chunks, taken
where there are few blocks, need more): the gradient of bem_vjp, whose sums differ in their order (1e-10 of the
largest entry, as for the float64 adjoint against the oracle)."""
import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu


def _need(K, M, N):
    """Bytes with the fewest chunks: blocks of at least 256 samples, about 4,096 of them."""
    def chunks(n, groups):
        c = max(1, min(-(-4096 // groups), -(-n // 256)))
        return max(1, -(-n // -(-n // c)))
    r = lambda b: -(-b // 256) * 256
    kg, mg = -(-K // 64), -(-M // 64)
    ns, ng, ne = chunks(N, kg), chunks(3 * M, kg), chunks(N, mg)
    return (r(K * 192) + r(K * 96) + r(M * 64) + r(M * 32) + r(M * 24) + r((ns + ng) * K * 128) +
            r((ne * M * 3 + 6 * M) * 8) + r(15 * M * 8) + r(K * 128))


@pytest.mark.parametrize("K,side,N", [(51136, 2, 5000), (51136, 2, 16384), (50911, 4, 50000), (50911, 4, 100000)])
def test_last_sizes(K, side, N):
    assert _need(K, 4 * side, N) <= 64 << 20 < _need(K + 1024, 4 * side, N)
    ctx = ctx_for(1, per_side=side, handle_model="straight")
    rng = np.random.default_rng(K)
    a = rng.uniform(0.1, 0.85, (K, 2))
    th = dev(np.concatenate([a, a + 0.004, W.draw_straight_colours(rng, K)], 1))
    x, g = dev(W.random_points(1, N, 0.01, 0.99)), dev(W.random_vector(2, (N, 3)))
    out = torch.empty_like(th)
    ctx.vjp_noalloc(th, x, g, out)
    want = host(ctx.vjp(th, x, g, "fp64"))
    assert np.abs(host(out) - want).max() < 1e-10 * np.abs(want).max()
    with pytest.raises(B.BemError):
        ctx.vjp_noalloc(torch.cat([th, th[:1024]]), x, g, torch.empty(K + 1024, 10, dtype=torch.float64, device="cuda"))
