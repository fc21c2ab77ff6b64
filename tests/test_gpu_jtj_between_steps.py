"""bem_jtj in split BF16 only enqueues after its first call of a configuration, also after an LM step over cells, whose
Gram has a work list of its own: an event behind work that is still running is pending when the call returns."""
import pytest
import torch

from paper_2602_05492_amd import bem as B
from paper_2602_05492_amd import workload as W
from helpers import ctx_for, dev

pytestmark = pytest.mark.gpu


def test_no_host_synchronisation():
    ctx, th = ctx_for(8), dev(W.random_handles(3, 40, spread=0.03))
    x = dev(W.random_points(4, 60000, 1e-3, 1 - 1e-3))
    T = ctx.eval(th, x, (0.3, 0.5, 0.7), "fp64") + 0.05 * dev(W.random_vector(5, (60000, 3)))
    r = dev(W.random_vector(6, (60000, 3)), torch.float32)
    J, g = ctx.jtj(th, x, r, "bf16x3_mfma", "mixed")
    for _ in range(2):
        ctx.profile(True)
        ctx.lm_step(th.clone(), x, T, B.new_lm_state(1.0), "bf16x3_mfma", "mixed")
        assert ctx.profile_read()["beta_rows"][1] == 0                  # over cells
        ctx.profile(False)
        torch.cuda.synchronize()
        torch.cuda._sleep(200_000_000)                                  # some 0.1 s
        ev = torch.cuda.Event()
        ev.record()
        J1, g1 = ctx.jtj(th, x, r, "bf16x3_mfma", "mixed")
        pending = not ev.query()
        torch.cuda.synchronize()
        assert pending
        assert float((J1 - J).abs().max()) <= 1e-6 * float(J.abs().max())
