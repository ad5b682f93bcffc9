"""The order of summation of the running sum and of the regression's tree, held to the bit.

The coefficients of a fit answer to the last bit of the R factors: the column-scaled problem is
solved to a few eps whatever the tree, but the coefficient vector itself is dominated by terms
whose share of the scaled solution is tiny, and two trees of the same quality give vectors that
differ by up to 1e-9 of its norm (the curve differs by 1e-9 at most and is checked against the
oracle elsewhere).  So the order of all sums is fixed, whatever kernel forms them: 16 entries, 256
of those, chunk after chunk; lanes by halves, four wavefronts, 256 rows a workgroup.

flodance_bits.txt holds what that order gives on gfx950 for pivots made by exact arithmetic
(uniform numbers, divisions), from the first kernels of this library that had it: one row per
thread, the sums by shuffles.  A line: n d n0 ns q seed, then ell at the places below and the
coefficients, as hexadecimal floats.
"""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
GOLDEN = os.path.join(HERE, "golden", "flodance_bits.txt")


def pivots(n, seed):
    u = np.random.default_rng(seed).random(n)
    return torch.from_numpy((0.75 + 0.5 * u) / (1.0 + np.arange(n) / 64.0)).cuda()


def places(n):
    return sorted({i for i in (0, 15, 16, 4095, 4096, n // 2, n - 1) if i < n})


def lines():
    with open(GOLDEN) as f:
        return [x.split() for x in f if x.strip()]


@pytest.mark.parametrize("line", lines(), ids=lambda x: "-".join(x[:6]))
def test_running_sum_and_coefficients(line):
    import paper_2503_04424_amd as M
    M.load()
    n, d, n0, ns, q, seed = map(int, line[:6])
    ell = M.mdet_principal_logdets(pivots(n, seed))
    coef = M.mdet_flodance_fit(ell, d, n0, ns, q)
    got = torch.cat([ell[places(n)], coef]).cpu().numpy()
    assert [float(x).hex() for x in got] == line[6:]
