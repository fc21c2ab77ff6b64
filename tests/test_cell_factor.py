"""The factor of a grid cell's Gramian (cell_factor.hpp), built for the host: R R^T = Phi Phi^T and R Q = Phi for cells
whose samples do and do not determine the 64 node functions.  Runs without a GPU.

Bars, floor = 1e-13 the largest pivot left out, relative to the largest diagonal entry `top` of Phi Phi^T: the remainder
of R R^T has diagonal entries of at most floor top (its others are smaller), and 64 steps of 64 x 64 products round at
64^2 2^-53 = 5e-13 at the worst: 1e-12 top.  What R Q leaves out of a node function has the remainder's diagonal entry
as its sum of squares over the samples, so at most sqrt(floor top) at any of them; Q's rounding (64 terms of at most
1 / sqrt(floor top) at 2^-53) adds less than 1e-7.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "hostmath", "cellfactor_host.cpp")
CSRC = os.path.join(HERE, "..", "paper_2602_05492_amd", "csrc")
HDRS = [os.path.join(CSRC, f) for f in ("cell_factor.hpp", "seg_math.hpp")]
LIB = os.path.join(HERE, "hostmath", "libcellfactor_host.so")


@pytest.fixture(scope="module")
def factor():
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(f) for f in [SRC, *HDRS]):
        subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", SRC, "-o", LIB], check=True, capture_output=True)
    L = ctypes.CDLL(LIB)
    L.hm_cell_factor.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    L.hm_pivot_floor.restype = ctypes.c_double

    def call(x):
        x = np.ascontiguousarray(x)
        R, C = np.zeros((64, 64)), np.zeros((64, 64))
        L.hm_cell_factor(x.ctypes.data, len(x), R.ctypes.data, C.ctypes.data)
        return R, C

    return call, L.hm_pivot_floor()


def _cheb(t, n):
    v = [np.ones_like(t), t]
    for _ in range(2, n):
        v.append(2 * t * v[-1] - v[-2])
    return np.array(v)


def _products(x):                          # T_a(xi) T_b(eta), row b 8 + a
    return np.einsum("bn,an->ban", _cheb(x[:, 1], 8), _cheb(x[:, 0], 8)).reshape(64, -1)


def _phi(x):                               # node functions at the samples, row j 8 + i
    a, i = np.arange(8)[:, None], np.arange(8)[None]
    d = np.cos(a * (2 * i + 1) * np.pi / 16) * np.where(a == 0, 1 / 8, 2 / 8)
    return np.kron(d.T, d.T) @ _products(x)


def _cut(rng, n, keep):
    u = rng.uniform(-1, 1, (200 * n, 2))
    return u[keep(u)][:n]


def _cell(kind, n, rng):
    u = rng.uniform(-1, 1, (n, 2))
    if kind == "uniform":
        return u
    if kind.startswith("triangle"):        # a corner, legs of a quarter of the width
        sx, sy = {"0": (1, 1), "1": (1, -1), "2": (-1, 1), "3": (-1, -1)}[kind[-1]]
        return _cut(rng, n, lambda v: (v * [sx, sy] + 1).sum(1) < 0.5)
    if kind == "diagonal":
        return _cut(rng, n, lambda v: v.sum(1) < 0)
    if kind.startswith("strip"):           # at each side
        k = int(kind[-1])
        u[:, k & 1] = (-1 + 0.3 * (u[:, k & 1] + 1)) * (1 if k < 2 else -1)
        return u
    if kind == "line":
        return np.outer(u[:, 0], [0.7, -0.4]) + [0.1, 0.3]
    if kind == "point":
        return np.clip(u[:1] + 1e-5 * u, -1, 1)
    if kind == "repeated":
        return u[np.arange(n) % (n // 5 + 1)]
    return np.sign(u) * np.where(rng.random((n, 2)) < 0.5, 1.0, np.abs(u))      # "edges"


KINDS = ["uniform", "triangle0", "triangle1", "triangle2", "triangle3", "diagonal", "strip0", "strip1", "strip2", "strip3",
         "line", "point", "repeated", "edges"]


@pytest.mark.parametrize("kind", KINDS)
def test_factor(factor, kind):
    call, floor = factor
    rng = np.random.default_rng(KINDS.index(kind))
    for n in [1, 2, 3, 5, 9, 20, 40, 63, 64, 65, 80, 100, 140, 600]:
        for _ in range(3):
            x = _cell(kind, n, rng)
            R, C = call(x)
            P = _phi(x)
            G = P @ P.T
            top = G.diagonal().max()
            Q = C @ _products(x)
            assert np.abs(R @ R.T - G).max() < 1e-12 * top, (kind, n)
            assert np.abs(R @ Q - P).max() < np.sqrt(floor * top) + 1e-7, (kind, n)
            assert np.abs(Q).max() < 1.01, (kind, n)
            rank = int((np.abs(R).max(0) > 0).sum())
            assert rank <= min(n, 64) and not R[:, rank:].any() and not C[rank:].any()
