"""Performance cases: the calls that programs using this library make, over the sizes they make them at.

A case is a dict of plain values; its `kind` names the call:
  eval     Context.eval            colours at N points (a preview, a rendered image, probe points)
  grad     bem_eval + backward     one gradient step's forward and adjoint on N samples
  jtj      Context.jtj             normal equations on N samples
  lm       Context.lm_step         one Levenberg-Marquardt step on N samples
  regions  lm_step_subdomains      one step in two regions of the image that a slanted edge separates
Sizes follow the library's workloads (4 to 256 cubic handles of 16 or 32 segments, 500 straight handles, 1,000 to
4,194,304 samples, 256 outer elements per side).

Mixed precision computes in float32, and the mixed cases are the programs that use it: their curve parameters and
their targets live in float32, torch's default, are widened for the call, and take its result back in float32.
The float64 cases keep everything in float64.

exact() evaluates the same formulas in plain torch float64: closed-form segment integrals of the regularised kernels,
the Galerkin boundary system with its smallest singular value dropped (from an SVD), derivatives by autograd, a dense
Cholesky solve.
"""
import math
import random

import numpy as np
import torch

from paper_2602_05492_amd import bem as B

EPS = 1e-2
PER_SIDE = 256
CBAR = (0.5, 0.45, 0.4)


# ---- the cases ------------------------------------------------------------------------------------------------
def _case(kind, model, H, S, N, prec, near=0.0, name=None):
    c = {"kind": kind, "model": model, "H": H, "S": S, "N": N, "prec": prec, "near": near}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a few curves looked at in a few points while a user drags a handle: launches and latency
        _case("eval", "cubic", 4, 32, 1000, "mixed", name="eval-probe"),
        # the 512 x 512 pixel grid of a mid-sized drawing, in reference precision
        _case("eval", "cubic", 32, 16, 512 * 512, "fp64", name="eval-grid-fp64"),
        # the paper's handle count on an image grid
        _case("eval", "straight", 500, 1, 512 * 512, "mixed", name="eval-straight"),
        # a large drawing at a million samples, a tenth of them hugging the curves
        _case("eval", "cubic", 128, 32, 1048576, "mixed", near=0.1, name="eval-near"),
        # gradient steps: a small scene in float64, the paper's handles on its 100,000 samples (an odd number of
        # them), the large adjoint workload
        _case("grad", "cubic", 4, 32, 16384, "fp64", name="grad-tiny-fp64"),
        _case("grad", "straight", 500, 1, 100003, "mixed", name="grad-straight"),
        _case("grad", "cubic", 256, 32, 4194304, "mixed", name="grad-large"),
        # normal equations of a small scene for a caller's own solver
        _case("jtj", "cubic", 4, 32, 16384, "fp64", name="jtj-tiny-fp64"),
        # LM steps: the medium workload in float64, the paper's setting, the LM workload
        _case("lm", "cubic", 32, 16, 262144, "fp64", name="lm-medium-fp64"),
        _case("lm", "straight", 500, 1, 100000, "mixed", name="lm-paper"),
        _case("lm", "cubic", 256, 32, 2097152, "mixed", name="lm-large"),
        # two regions with their own boundaries, handles and compatible steps (the paper's subdomains)
        _case("regions", "straight", 60, 1, 30000, "mixed", name="lm-regions"),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; every second one odd."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.5 else n))


def draw(rng: random.Random):
    kind = rng.choice(["eval", "eval", "grad", "grad", "jtj", "lm", "lm", "regions"])
    model = "straight" if kind == "regions" or rng.random() < 0.35 else "cubic"
    prec = "mixed" if kind == "regions" else rng.choice(["mixed", "mixed", "fp64"])
    S = 1 if model == "straight" else rng.choice([8, 16, 32])
    H = _log_int(rng, 4, 500 if model == "straight" else 256)
    near = rng.choice([0.0, 0.0, 0.1]) if kind in ("eval", "grad") else 0.0
    top = {"eval": 1048576, "grad": 1048576, "jtj": 65536, "lm": 262144, "regions": 131072}[kind]
    if prec == "fp64":
        top = min(top, 131072)
        H = min(H, 100)
    if kind == "jtj":
        prec, H = "fp64", min(H, 48)
    if kind == "regions":
        H = min(H, 200)
    return _case(kind, model, H, S, _log_int(rng, 1000, top), prec, near)


# ---- inputs ---------------------------------------------------------------------------------------------------
def _theta(case, g, H, lo=(0.15, 0.15), hi=(0.85, 0.85)):
    """Handles in a box: cubic curves whose spread shrinks with their number (about a fifth of the pairs cross), or
    straight handles of a twentieth of the image; colour jumps of left and right colours in [0, 1]."""
    lo, hi = torch.tensor(lo, dtype=torch.float64), torch.tensor(hi, dtype=torch.float64)

    def rand(*s):
        return torch.rand(*s, generator=g, dtype=torch.float64)

    centre = lo + (hi - lo) * rand(H, 1, 2)
    if case["model"] == "straight":
        ang = 2 * math.pi * rand(H, 1)
        a = centre[:, 0]
        ends = torch.cat([a, torch.minimum(torch.maximum(a + 0.05 * torch.cat([ang.cos(), ang.sin()], 1), lo), hi)], 1)
        c = rand(H, 2, 3)
        return torch.cat([ends, c[:, 0] - c[:, 1], c[:, 0] + c[:, 1] - 1.0], 1)
    spread = min(0.5, 0.38 * math.sqrt(32 / H))
    ctrl = torch.minimum(torch.maximum(centre + spread * (2 * rand(H, 4, 2) - 1), lo), hi)
    c = rand(H, 2, 2, 3)
    wd, wc = c[:, :, 0] - c[:, :, 1], c[:, :, 0] + c[:, :, 1] - 1.0
    return torch.cat([ctrl.reshape(H, 8), wd.reshape(H, 6), wc.reshape(H, 6)], 1)


def _samples(case, theta, g, dev):
    """Uniform samples of the unit square; a share `near` of them within 1e-3 of a handle."""
    N = case["N"]
    x = torch.rand(N, 2, generator=g, dtype=torch.float64, device=dev).clamp_(1e-7, 1 - 1e-7)
    k = int(round(case["near"] * N))
    if k:
        a, b = (v.to(dev) for v in _polyline(theta, case["S"])[:2])
        i = torch.randint(0, len(a), (k,), generator=g, device=dev)
        r = torch.rand(k, 2, generator=g, dtype=torch.float64, device=dev)
        v = b[i] - a[i]
        n = torch.stack([v[:, 1], -v[:, 0]], 1) / v.norm(dim=1, keepdim=True).clamp_min(1e-12)
        x[N - k:] = a[i] + r[:, :1] * v + 2e-3 * (r[:, 1:] - 0.5) * n
    return x


def _targets(x, g):
    """A smooth colour image with noise: what a renderer's samples look like to the fit."""
    c = torch.rand(3, 4, generator=g, dtype=torch.float64, device=x.device)
    img = 0.5 + 0.3 * torch.sin(2 * math.pi * (x @ (3 * c[:, :2]).T + c[:, 2])) * c[:, 3]
    return img + 0.2 * torch.randn(img.shape, generator=g, dtype=torch.float64, device=x.device)


def _region_polygons():
    return [[(0.0, 0.0), (0.6, 0.0), (0.4, 1.0), (0.0, 1.0)], [(0.6, 0.0), (1.0, 0.0), (1.0, 1.0), (0.4, 1.0)]]


def _elements(poly, length=1.0 / 128):
    out = []
    for p, q in zip(poly, poly[1:] + poly[:1]):
        p, q = np.array(p), np.array(q)
        n = int(math.ceil(np.linalg.norm(q - p) / length))
        t = (np.arange(n + 1) / n)[:, None]
        v = p * (1 - t) + q * t
        out.append(np.concatenate([v[:-1], v[1:]], 1))
    return np.concatenate(out)


def _inputs(case, seed, dev):
    """Everything drawn from the seed, in float64: handles, samples, targets and (regions) labels."""
    g = torch.Generator().manual_seed(1000003 * seed + 17)
    gd = torch.Generator(device=dev).manual_seed(1000003 * seed + 29)
    d = {}
    if case["kind"] == "regions":
        d["thetas"] = [_theta(case, g, case["H"], (0.05, 0.05), (0.38, 0.95)),
                       _theta(case, g, case["H"], (0.62, 0.05), (0.95, 0.95))]
        d["x"] = _samples(case, None, gd, dev)
        d["labels"] = (d["x"][:, 0] > 0.6 - 0.2 * d["x"][:, 1]).to(torch.int32)
    else:
        d["theta"] = _theta(case, g, case["H"])
        d["x"] = _samples(case, d["theta"], gd, dev)
    if case["kind"] in ("grad", "lm", "regions"):
        d["T"] = _targets(d["x"], gd)
    if case["kind"] == "jtj":
        d["r"] = torch.randn(d["x"].shape[0], 3, generator=gd, dtype=torch.float64, device=dev)
    if case["prec"] == "mixed":          # what a float32 program holds
        for k in ("theta", "T"):
            if k in d:
                d[k] = d[k].float().double()
        if "thetas" in d:
            d["thetas"] = [t.float().double() for t in d["thetas"]]
    return d


def _lambda(case):
    """Damping at which a step from these parameters is usually accepted."""
    return 1.0 if case["model"] == "straight" else 0.1


# ---- one pass -------------------------------------------------------------------------------------------------
class _State:
    pass


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    d = _inputs(case, seed, dev)
    s = _State()
    s.kind, s.prec, s.lam = case["kind"], case["prec"], _lambda(case)
    s.gram = "bf16x3_mfma" if s.prec == "mixed" else "fp64"
    own = torch.float32 if s.prec == "mixed" else torch.float64
    kw = dict(segs_per_handle=case["S"], eps=EPS, handle_model=case["model"])
    if s.kind == "regions":
        s.ctxs = [B.Context(elements=_elements(p), **kw) for p in _region_polygons()]
        s.params = [t.to(dev, own) for t in d["thetas"]]
        s.labels = d["labels"]
    else:
        s.ctx = B.Context(elems_per_side=PER_SIDE, **kw)
        s.theta = d["theta"].to(dev)
        if s.kind in ("grad", "lm"):
            s.param = s.theta.to(own).requires_grad_(s.kind == "grad")
    s.x = d["x"]
    if s.kind == "grad":
        s.T = d["T"].to(own)
    elif "T" in d:
        s.T = d["T"]
    if s.kind == "jtj":
        s.r = d["r"]
    return s


def run(s):
    if s.kind == "eval":
        return s.ctx.eval(s.theta, s.x, CBAR, s.prec)
    if s.kind == "grad":
        s.param.grad = None
        u = B.bem_eval(s.param.double(), s.x, s.ctx, CBAR, s.prec)
        torch.nn.functional.mse_loss(u, s.T).backward()
        return {"u": u.detach(), "grad": s.param.grad}
    if s.kind == "jtj":
        JtJ, Jtr = s.ctx.jtj(s.theta, s.x, s.r, s.gram, s.prec)
        return {"JtJ": JtJ, "Jtr": Jtr}
    if s.kind == "lm":
        th = s.param.to(torch.float64, copy=True)
        st = B.new_lm_state(s.lam)
        s.ctx.lm_step(th, s.x, s.T, st, s.gram, s.prec)
        out = {"theta": th.to(s.param.dtype), "cbar": list(st.cbar), "accepted": st.accepted}
        if s.prec == "fp64":
            out["loss"] = [st.loss_before, st.loss_after]
        return out
    ths = [p.to(torch.float64, copy=True) for p in s.params]
    sts = [B.new_lm_state(s.lam, compat=1) for _ in s.ctxs]
    B.lm_step_subdomains(s.ctxs, ths, s.x, s.T, s.labels, sts, s.gram, s.prec)
    return {"thetas": [t.to(s.params[0].dtype) for t in ths], "cbar": [list(t.cbar) for t in sts],
            "accepted": [t.accepted for t in sts]}


def work(case):
    """Bytes of the inputs and outputs, and the floating-point operations of the direct closed-form sums: about 110
    a sample and segment forward (40 an outer element), twice that again for the adjoint, 500 a pair of a Jacobian row,
    two an entry and sample of the augmented Gram matrix, P^3 / 3 of the Cholesky."""
    H, S, N = case["H"], case["S"], case["N"]
    Q, G, C = (10, 4, 2) if case["model"] == "straight" else (20, 8, 4)
    M, K = 4 * PER_SIDE, H * S
    if case["kind"] == "regions":
        M = 430
    P = Q * H
    e = 4 if case["prec"] == "mixed" else 8
    fwd = N * (110.0 * K + 40.0 * M)
    b, f = 16.0 * N + 8.0 * P, fwd
    if case["kind"] == "eval":
        return {"bytes": b + 3 * e * N, "flops": f}
    if case["kind"] == "grad":
        return {"bytes": b + 6 * e * N + e * P, "flops": 3 * f}
    area = 3 * (G * H) ** 2 / 2 + 3 * G * H * (C * H + M) + (C * H + M) ** 2 / 2
    f = 500.0 * N * K + 2.0 * N * area
    if case["kind"] == "jtj":
        return {"bytes": b + 24.0 * N + 8.0 * (P * P + P), "flops": f}
    f += 2 * fwd + P ** 3 / 3.0 * (2 if case["kind"] == "regions" else 1)
    return {"bytes": b + 24.0 * N + e * P, "flops": f}


# ---- the same in plain float64 torch --------------------------------------------------------------------------
def _bernstein(t):
    return torch.stack([(1 - t) ** 3, 3 * (1 - t) ** 2 * t, 3 * (1 - t) * t ** 2, t ** 3], 1)


def _weights(theta, S):
    """Vertex weights on the geometry parameters [S + 1, G / 2] and on the jumps at either end [S + 1, 1 or 2]."""
    t = torch.arange(S + 1, dtype=theta.dtype, device=theta.device) / S
    if theta.shape[1] == 10:
        return torch.stack([1 - t, t], 1), torch.ones_like(t)[:, None]
    return _bernstein(t), torch.stack([1 - t, t], 1)


def _polyline(theta, S):
    """Segment end points a, b [K, 2] and end densities wd_a, wd_b, wc_a, wc_b [K, 3]."""
    Wg, Wj = _weights(theta, S)
    g, j = 2 * Wg.shape[1], Wj.shape[1]
    H = theta.shape[0]
    p = (Wg @ theta[:, :g].reshape(H, -1, 2))
    wd = Wj @ theta[:, g:g + 3 * j].reshape(H, j, 3)
    wc = Wj @ theta[:, g + 3 * j:].reshape(H, j, 3)
    return tuple(v[:, sl].reshape(-1, v.shape[2]) for v in (p, wd, wc) for sl in (slice(0, S), slice(1, S + 1)))


def _moments(x, ax, ay, bx, by, eps):
    """Double- and single-layer integrals of the two hat functions of segments a -> b seen from x [n, 2]."""
    X, Y = x[:, :1], x[:, 1:]
    vx, vy = bx - ax, by - ay
    L = (vx * vx + vy * vy).sqrt()
    tx, ty = vx / L, vy / L
    t0 = (X - ax) * tx + (Y - ay) * ty
    h = (ax - X) * ty - (ay - Y) * tx
    u1 = L - t0
    q2 = h * h + eps * eps
    q = q2.sqrt()
    r0, r1 = t0 * t0 + q2, u1 * u1 + q2
    l0, ell = r0.log(), torch.log1p(L * (u1 - t0) / r0)
    D = torch.atan2(q * L, q2 - t0 * u1)
    K0d, K1d = h / q * D / (2 * math.pi), h * ell / (4 * math.pi)
    K0s = -(u1 * ell + L * l0 - 2 * L + 2 * q * D) / (4 * math.pi)
    K1s = -(r1 * ell + L * (u1 - t0) * (l0 - 1)) / (8 * math.pi)
    db, sb = (K1d + t0 * K0d) / L, (K1s + t0 * K0s) / L
    return K0d - db, db, K0s - sb, sb


def _chunks(n, k, pairs=1 << 22):
    step = max(1, pairs // max(k, 1))
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _handle_term(x, seg):
    a, b, wda, wdb, wca, wcb = seg
    out = []
    for sl in _chunks(len(x), len(a)):
        da, db, sa, sb = _moments(x[sl], a[:, 0], a[:, 1], b[:, 0], b[:, 1], EPS)
        out.append(da @ wda + db @ wdb + sa @ wca + sb @ wcb)
    return torch.cat(out)


def _handle_grad(x, g, theta, S):
    """Gradient of sum_x g(x) . f(x) with respect to theta."""
    total = torch.zeros_like(theta)
    for sl in _chunks(len(x), theta.shape[0] * S):
        th = theta.clone().requires_grad_()
        a, b, wda, wdb, wca, wcb = _polyline(th, S)
        da, db, sa, sb = _moments(x[sl], a[:, 0], a[:, 1], b[:, 0], b[:, 1], EPS)
        total += torch.autograd.grad((g[sl] * (da @ wda + db @ wdb + sa @ wca + sb @ wcb)).sum(), th)[0]
    return total


def _handle_jacobian(x, theta, S):
    """df_c(x)/dtheta [n, 3, H, Q] for one chunk of samples."""
    n, H = len(x), theta.shape[0]
    Wg, Wj = _weights(theta, S)
    a, b, wda, wdb, wca, wcb = _polyline(theta, S)
    end = [v.expand(n, -1).clone().requires_grad_() for v in (a[:, 0], a[:, 1], b[:, 0], b[:, 1])]
    mom = _moments(x, *end, EPS)
    J = torch.zeros(n, 3, H, theta.shape[1], dtype=x.dtype, device=x.device)
    G, j = 2 * Wg.shape[1], Wj.shape[1]
    for c in range(3):
        f = mom[0] * wda[:, c] + mom[1] * wdb[:, c] + mom[2] * wca[:, c] + mom[3] * wcb[:, c]
        gr = [v.reshape(n, H, S) for v in torch.autograd.grad(f.sum(), end, retain_graph=True)]
        J[:, c, :, 0:G:2] = gr[0] @ Wg[:-1] + gr[2] @ Wg[1:]
        J[:, c, :, 1:G:2] = gr[1] @ Wg[:-1] + gr[3] @ Wg[1:]
    m = [v.detach().reshape(n, H, S) for v in mom]
    for k, (p, q) in enumerate(((m[0], m[1]), (m[2], m[3]))):
        col = p @ Wj[:-1] + q @ Wj[1:]
        for e in range(j):
            for c in range(3):
                J[:, c, :, G + 3 * (j * k + e) + c] = col[:, :, e]
    return J


class _Boundary:
    """Outer elements, their Gauss points and weights, and the pseudo-inverse without the smallest singular value."""

    def __init__(self, elems, dev):
        e = torch.as_tensor(elems, dtype=torch.float64)
        a, b = e[:, :2], e[:, 2:]
        mid, half = (a + b) / 2, (b - a) / 2
        node = torch.tensor([-math.sqrt(0.6), 0.0, math.sqrt(0.6)], dtype=torch.float64)
        ln = half.norm(dim=1)
        gp = (mid[:, None] + node[:, None] * half[:, None]).reshape(-1, 2)
        gw = (torch.tensor([5 / 9, 8 / 9, 5 / 9], dtype=torch.float64) * ln[:, None]).reshape(-1)
        nrm = torch.stack([half[:, 1], -half[:, 0]], 1) / ln[:, None]
        M = len(e)
        d = gp[None] - gp[:, None]
        r2 = (d * d).sum(-1)
        k = -(d * nrm.repeat_interleave(3, 0)[None]).sum(-1) / (2 * math.pi * r2)
        own = torch.arange(M).repeat_interleave(3)
        k = torch.where(own[:, None] == own[None], torch.zeros_like(k), k) * gw[:, None] * gw
        A = k.reshape(M, 3, M, 3).sum((1, 3)) + torch.diag(ln)
        u, s, vt = np.linalg.svd(A.numpy())
        self.pinv = torch.from_numpy((vt[:-1].T / s[:-1]) @ u[:, :-1].T).to(dev)
        self.a, self.b, self.gp, self.gw, self.M = a.to(dev), b.to(dev), gp.to(dev), gw.to(dev), M

    def values(self, seg):
        f = _handle_term(self.gp, seg) * self.gw[:, None]
        return self.pinv @ f.reshape(self.M, 3, 3).sum(1)

    def beta(self, x):
        d, e = self.a[None] - x[:, None], self.b[None] - x[:, None]
        return torch.atan2(d[..., 0] * e[..., 1] - d[..., 1] * e[..., 0], (d * e).sum(-1)) / (2 * math.pi)

    def apply(self, x, U):
        return torch.cat([self.beta(x[sl]) @ U for sl in _chunks(len(x), self.M)])


def _square():
    c = [(0.0, 0.0), (1.0, 0.0), (1.0, 1.0), (0.0, 1.0)]
    return _elements(c, 1.0 / PER_SIDE)


def _colours(x, theta, S, bnd, cbar):
    seg = _polyline(theta, S)
    return torch.as_tensor(cbar, dtype=torch.float64, device=x.device) + bnd.apply(x, bnd.values(seg)) + _handle_term(x, seg)


def _normal_equations(x, r, theta, S, bnd, m):
    """(1/m) sum J^T J and J^T r."""
    P = theta.numel()
    Fg = torch.zeros(bnd.M, 3 * P, dtype=torch.float64, device=x.device)
    for sl in _chunks(bnd.M, 3 * theta.shape[0] * S):
        q = slice(3 * sl.start, 3 * sl.stop)
        J = _handle_jacobian(bnd.gp[q], theta, S) * bnd.gw[q, None, None, None]
        Fg[sl] = J.reshape(-1, 3, 3 * P).sum(1)
    Z = bnd.pinv @ Fg
    H = torch.zeros(P, P, dtype=torch.float64, device=x.device)
    g = torch.zeros(P, dtype=torch.float64, device=x.device)
    for sl in _chunks(len(x), max(theta.shape[0] * S, bnd.M, P)):
        J = _handle_jacobian(x[sl], theta, S).reshape(-1, 3 * P) + bnd.beta(x[sl]) @ Z
        J = J.reshape(-1, P)
        H += J.T @ J
        g += J.T @ r[sl].reshape(-1)
    return H / m, g / m


def _flux(theta):
    """Columns a_c [P, 3] of the flux condition of straight handles: the handle's length at its wc."""
    A = torch.zeros(theta.shape[0], 10, 3, dtype=torch.float64, device=theta.device)
    ln = (theta[:, 2:4] - theta[:, :2]).norm(dim=1)
    for c in range(3):
        A[:, 7 + c, c] = ln
    return A.reshape(-1, 3)


def _step(x, T, theta, S, bnd, lam, m, compat):
    """One damped step: (theta', mean colour, accepted, losses)."""
    cbar = T.mean(0)
    r = _colours(x, theta, S, bnd, cbar) - T
    L0 = float((r * r).sum()) / (2 * m)
    H, g = _normal_equations(x, r, theta, S, bnd, m)
    d = torch.diag(H)
    Hd = (H + lam * torch.diag(torch.maximum(d, 1e-12 * d.max()))).cpu()
    ch = torch.linalg.cholesky(Hd)
    step = torch.cholesky_solve(g.cpu()[:, None], ch).to(x.device)
    if compat:
        A = _flux(theta)
        Y = torch.cholesky_solve(A.cpu(), ch).to(x.device)
        step = step - Y @ torch.linalg.solve(A.T @ Y, A.T @ step)
    new = theta - step.reshape(theta.shape)
    if compat:
        A, flat = _flux(new), new.reshape(-1)
        new = (flat - A @ ((A.T @ flat) / (A * A).sum(0))).reshape(theta.shape)
    r = _colours(x, new, S, bnd, cbar) - T
    L1 = float((r * r).sum()) / (2 * m)
    ok = L1 < L0
    return (new if ok else theta), cbar.tolist(), int(ok), [L0, L1]


def exact(case, seed):
    pairs = float(case["N"]) * (case["H"] * case["S"] + 4 * PER_SIDE)
    if pairs > {"eval": 8e9, "grad": 2e9}.get(case["kind"], 5e8):
        return None
    dev = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
    d = _inputs(case, seed, dev)
    x, S = d["x"], case["S"]
    if case["kind"] == "regions":
        out = {"thetas": [], "cbar": [], "accepted": []}
        for k, (poly, th) in enumerate(zip(_region_polygons(), d["thetas"])):
            keep = d["labels"] == k
            t, c, ok, _ = _step(x[keep], d["T"][keep], th.to(dev), S, _Boundary(_elements(poly), dev), _lambda(case), len(x), True)
            out["thetas"].append(t)
            out["cbar"].append(c)
            out["accepted"].append(ok)
        return out
    theta, bnd = d["theta"].to(dev), _Boundary(_square(), dev)
    if case["kind"] == "eval":
        return _colours(x, theta, S, bnd, CBAR)
    if case["kind"] == "grad":
        u = _colours(x, theta, S, bnd, CBAR)
        g = 2 * (u - d["T"]) / u.numel()
        psi = torch.zeros(bnd.M, 3, dtype=torch.float64, device=dev)
        for sl in _chunks(len(x), bnd.M):
            psi += bnd.beta(x[sl]).T @ g[sl]
        mu = (bnd.pinv.T @ psi).repeat_interleave(3, 0) * bnd.gw[:, None]
        return {"u": u, "grad": _handle_grad(x, g, theta, S) + _handle_grad(bnd.gp, mu, theta, S)}
    if case["kind"] == "jtj":
        H, g = _normal_equations(x, d["r"], theta, S, bnd, len(x))
        return {"JtJ": H, "Jtr": g}
    t, c, ok, loss = _step(x, d["T"], theta, S, bnd, _lambda(case), len(x), False)
    out = {"theta": t, "cbar": c, "accepted": ok}
    if case["prec"] == "fp64":
        out["loss"] = loss
    return out
