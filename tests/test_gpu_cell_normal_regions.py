"""J^T J over grid cells where samples do not fill the cells: regions with a slanted edge, samples on one side of a line,
in strips, in triangles and few to a cell.  Against the FP64 step: accepted at the given damping without a
retry, within helpers.mixed_step_tol.  That the cells' form was taken is read from the kernel families timed (the tiles
of samples have beta rows of their own).
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
REGIONS = [[(0.0, 0.0), (0.6, 0.0), (0.4, 1.0), (0.0, 1.0)], [(0.6, 0.0), (1.0, 0.0), (1.0, 1.0), (0.4, 1.0)]]


def _elements(poly, length=1.0 / 128):
    out = []
    for p, q in zip(poly, poly[1:] + poly[:1]):
        p, q = np.array(p), np.array(q)
        n = int(np.ceil(np.linalg.norm(q - p) / length))
        v = p + (np.arange(n + 1) / n)[:, None] * (q - p)
        out.append(np.concatenate([v[:-1], v[1:]], 1))
    return np.concatenate(out)


def _straight(seed, H, lo, hi, length=0.05):
    rng = np.random.default_rng(np.random.SeedSequence(entropy=9000 + seed))
    a = rng.uniform(lo, hi, size=(H, 2))
    ang = rng.uniform(0, 2 * np.pi, size=H)
    b = np.clip(a + length * np.stack([np.cos(ang), np.sin(ang)], 1), lo, hi)
    return np.ascontiguousarray(np.concatenate([a, b, W.draw_straight_colours(rng, H)], axis=1))


def _step(ctx, th0, x, T, gram, prec):
    th, st = th0.clone(), B.new_lm_state(LAM, 0)
    ctx.lm_step(th, x, T, st, gram, prec)
    return host(th - th0).ravel(), st


def _check(ctx, theta, x):
    th0, xd = dev(theta), dev(x)
    T = ctx.eval(th0, xd, CBAR, "fp64") + 0.05 * dev(W.random_vector(71, (len(x), 3)))
    d64, s64 = _step(ctx, th0, xd, T, "fp64", "fp64")
    ctx.profile(True)
    d, st = _step(ctx, th0, xd, T, "bf16x3_mfma", "mixed")
    ran = {k: launches for k, (_, launches) in ctx.profile_read().items()}
    ctx.profile(False)
    assert ran["beta_rows"] == 0 and ran["gram_mfma"] > 0
    JtJ, _ = ctx.jtj(th0, xd, torch.zeros_like(T), "fp64", "fp64")
    tol = mixed_step_tol(host(JtJ), LAM)
    e = np.abs(d - d64).max() / np.abs(d64).max()
    log(f"H={len(theta)} N={len(x)}: {e:.2e}, bar {tol:.2e}, retries {st.chol_retries}")
    assert s64.accepted == st.accepted == 1 and st.chol_retries == 0
    assert e < tol
    assert abs(st.loss_after - s64.loss_after) < 1e-5 * s64.loss_after


@pytest.mark.parametrize("H", [50, 200])
@pytest.mark.parametrize("d", [0, 1])
def test_region_with_a_slanted_edge(d, H):
    ctx = B.Context(segs_per_handle=1, elements=_elements(REGIONS[d]), handle_model="straight")
    x = W.random_points(30 + H + d, 140000, 1e-3, 1 - 1e-3)
    x = x[(x[:, 0] > 0.6 - 0.2 * x[:, 1]) == (d == 1)][:65000]
    _check(ctx, _straight(H + d, H, (0.05, 0.05) if d == 0 else (0.62, 0.05), (0.38, 0.95) if d == 0 else (0.95, 0.95)), x)
    ctx.close()


def _masked(kind, n, seed):
    x = W.random_points(seed, 12 * n, 1e-3, 1 - 1e-3)
    f = (x * 14) % 1.0                                   # place in a cell of some 1/14
    keep = {"line": x[:, 0] + 0.37 * x[:, 1] > 0.6,
            "low strips": (f < 0.3).any(1),              # strips at the lower and left sides
            "triangles": f.sum(1) < 0.6}[kind]
    return x[keep][:n]


@pytest.mark.parametrize("kind", ["line", "low strips", "triangles"])
@pytest.mark.parametrize("model", ["straight", "cubic"])
def test_samples_in_part_of_the_cells(kind, model):
    ctx = ctx_for(1 if model == "straight" else 16, handle_model=model)
    th = _straight(7, 120, 0.15, 0.85, 0.03) if model == "straight" else W.random_handles(7, 40, spread=0.03)
    _check(ctx, th, _masked(kind, 60000, 40))


def test_few_samples_in_most_cells():
    """15,000 samples in a ninth of the square, and cells elsewhere of 1 to 60."""
    x = 0.05 + W.random_points(50, 60000, 1e-3, 1 - 1e-3) / 3
    rest = W.random_points(51, 6000, 1e-3, 1 - 1e-3)
    rest = rest[rest[:, 0] ** 2 > W.random_points(52, len(rest), 0.0, 1.0)[:, 0]]      # from none to twice as many
    x[:: len(x) // len(rest)][: len(rest)] = rest
    _check(ctx_for(1, handle_model="straight"), _straight(9, 150, 0.05, 0.95, 0.03), x)


def test_regions_side_by_side():
    """The subdomains' call on both regions, with the compatibility condition, against its FP64 steps."""
    ctxs = [B.Context(segs_per_handle=1, elements=_elements(p), handle_model="straight") for p in REGIONS]
    ths = [dev(_straight(60, 80, (0.05, 0.05), (0.38, 0.95))), dev(_straight(61, 80, (0.62, 0.05), (0.95, 0.95)))]
    x = dev(W.random_points(62, 120000, 1e-3, 1 - 1e-3))
    labels = (x[:, 0] > 0.6 - 0.2 * x[:, 1]).to(torch.int32)
    T = 0.5 + 0.2 * dev(W.random_vector(63, (len(x), 3)))
    out = []
    for gram, prec in [("fp64", "fp64"), ("bf16x3_mfma", "mixed")]:
        th, st = [t.clone() for t in ths], [B.new_lm_state(LAM, compat=1) for _ in ths]
        B.lm_step_subdomains(ctxs, th, x, T, labels, st, gram, prec)
        assert [s.accepted for s in st] == [1, 1] and [s.chol_retries for s in st] == [0, 0]
        out.append([host(t) for t in th])
    for d in range(2):
        JtJ, _ = ctxs[d].jtj(ths[d], x[labels == d].contiguous(), torch.zeros_like(T[labels == d]), "fp64", "fp64")
        a, b = (o[d] - host(ths[d]) for o in out)
        e, tol = np.abs(a - b).max() / np.abs(a).max(), mixed_step_tol(host(JtJ), LAM)
        log(f"region {d}: {e:.2e}, bar {tol:.2e}")
        assert e < tol
        ctxs[d].close()
