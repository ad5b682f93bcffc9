"""The comparison that the GPU tests of pivoting use (separated.py) on the CPU: an elimination in numpy
in the tested precision passes it, and one with a mistake planted does not."""
from types import SimpleNamespace

import numpy as np
import pytest

import separated


def eliminate(a, order, group):
    """(pivots, factor as the library stores it) in a's own precision."""
    x = a[np.ix_(order, order)].copy()
    n = len(order)
    for j in range(n):
        l = x[j + 1:, j] / x[j, j]
        x[j + 1:, j + 1:] -= np.outer(l, x[j, j + 1:])
        x[j + 1:, j] = l
    stored = x.astype(np.float64)
    for g0 in range(group, n, group):
        g1 = min(n, g0 + group)
        stored[order[g0:g1], :g0] = x[g0:g1, :g0]
    return np.diag(x).astype(np.float64), stored


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,group", [(2, 64), (17, 64), (64, 64), (193, 64), (300, 128), (640, 512)])
def test_a_planted_mistake_is_seen(n, group, dtype):
    a = separated.matrix(n, dtype)
    o = separated.expected(a, group, dtype)
    r = SimpleNamespace(status=0, sign=o.sign, negative_pivots=o.negative_pivots)
    d, f = eliminate(a, o.perm, group)
    separated.check(o, group, dtype, r, d, o.perm, f)
    wrong = [(np.diag(a).astype(np.float64)[o.perm], f)]            # no multiplier applied
    i, j = n - 1, 0
    g = f.copy()
    g[i, j] = -g[i, j]                                              # one multiplier
    wrong.append((d, g))
    if n > 64:
        g = f.copy()
        g[:, [3, 40]] = g[:, [40, 3]]                               # two columns gathered the wrong way round
        wrong.append((d, g))
    for dd, ff in wrong:
        with pytest.raises(AssertionError):
            separated.check(o, group, dtype, r, dd, o.perm, ff)
