"""Float64 colours without handles are the mean colour at every finite sample, also where the squared distance to the
boundary overflows: an element seen from there subtends no angle."""
import numpy as np
import pytest

from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [130, 100003])
def test_no_handles(n):
    ctx, cbar = ctx_for(1), (0.3, 0.5, 0.7)
    x = W.random_points(3, n, 0.01, 0.99)
    far = [(1e200, 0.3), (-1e200, 0.3), (0.4, 1e180), (0.4, -1e307), (1e160, -1e160), (1e155, 1e154), (1e100, 1.0)]
    x[7:7 + 9 * len(far):9] = far
    x[64:128] = (2e154, 0.5)                                    # a wavefront of them
    u = host(ctx.eval(dev(np.zeros((0, 20))), dev(x), cbar, "fp64"))
    assert (u == np.array(cbar)).all()
