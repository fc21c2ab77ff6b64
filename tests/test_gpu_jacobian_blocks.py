"""bem_jacobian in blocks of samples: rows at the blocks' edges are those of a call on them alone (sums of the same
terms, their order by the size of the product: 1e-12 of the largest entry), and the workspace is the features and a
block of the rest, not a second copy of every sample's outer elements."""
import numpy as np
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16383, 16384, 16385, 40001])
def test_rows(n):
    ctx = B.Context(segs_per_handle=4, elems_per_side=16)
    th, x = dev(W.random_handles(3, 3)), dev(W.random_points(n, n, 0.01, 0.99))
    J = ctx.jacobian(th, x)
    for i in (0, 16380, n - 7, 32765):
        if i < n:
            r = ctx.jacobian(th, x[i:i + 9].contiguous())
            assert float((J[i:i + 9] - r).abs().max()) < 1e-12 * float(J.abs().max())
    ctx.close()


def test_workspace():
    n, M, nf = 200000, 1024, 3 * 8 + 4
    ctx = B.Context(segs_per_handle=1, handle_model="straight")
    th = dev(np.array([[0.3, 0.3, 0.4, 0.35, 0.1, 0.2, 0.3, 0.1, 0.0, 0.2], [0.6, 0.5, 0.7, 0.65, 0.3, 0.2, 0.1, 0.0, 0.1, 0.2]]))
    x = dev(W.random_points(4, n, 0.01, 0.99))
    ctx.jacobian(th, x[:1000].contiguous())
    torch.cuda.synchronize()
    out = torch.empty(n * 60, dtype=torch.float64, device="cuda")     # J's memory, of the caching allocator
    free = torch.cuda.mem_get_info()[0]
    del out
    ctx.jacobian(th, x)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert used < (M + nf) * n * 8 + nf * n * 8 + (256 << 20)
    ctx.close()
