"""lm_step_subdomains takes thetas and states as any iterables, as many steps as the shortest argument has (runs without
a GPU: contexts that record their calls)."""
import itertools
from types import SimpleNamespace

import pytest

from paper_2602_05492_amd import bem as B


class _Recorder:
    def __init__(self, calls):
        self.calls = calls

    def partition(self, labels, x, target, D):
        return list(x), list(target), [0, 2, 3, 6][: D + 1]

    def lm_step(self, theta, x, target, state, gram, prec):
        self.calls.append((self, theta, x, target, state, gram, prec))


class _X(list):
    shape = (6, 2)


def _state():
    return SimpleNamespace(data_count=0)


@pytest.mark.parametrize("wrap", [list, tuple, iter, lambda v: (a for a in v), lambda v: dict(enumerate(v)).values()])
def test_iterables(wrap):
    calls = []
    ctxs, thetas, sts = [_Recorder(calls) for _ in range(3)], ["t0", "t1", "t2"], [_state() for _ in range(3)]
    given = wrap(sts)
    out = B.lm_step_subdomains(ctxs, wrap(thetas), _X(range(6)), list("abcdef"), None, given, "fp64", "mixed")
    assert out is given
    assert [(c[0], c[1], c[2], c[3]) for c in calls] == [
        (ctxs[0], "t0", [0, 1], ["a", "b"]), (ctxs[1], "t1", [2], ["c"]), (ctxs[2], "t2", [3, 4, 5], ["d", "e", "f"])]
    assert all(c[4] is s and s.data_count == 6 for c, s in zip(calls, sts))
    assert all(c[5:] == ("fp64", "mixed") for c in calls)


def test_as_many_as_the_shortest():
    calls, st = [], _state()
    ctxs = [_Recorder(calls) for _ in range(3)]
    B.lm_step_subdomains(ctxs, ["t0", "t1"], _X(range(6)), list("abcdef"), None, itertools.repeat(st))
    assert [c[1] for c in calls] == ["t0", "t1"]
    B.lm_step_subdomains(ctxs, [], _X(range(6)), list("abcdef"), None, [])
    assert len(calls) == 2
