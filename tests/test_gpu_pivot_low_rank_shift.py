"""Blocks of low rank plus a small shift, whose Schur complement is far smaller than their entries: the forms that
look for pivots reduce an entry term by term from its value on, so that late roundings are relative to what is left
of it.  Sums that begin at zero and meet at the end (even and odd terms apart, say) round to the size of the entries."""
import numpy as np
import pytest
import torch

import paper_2503_04424_amd as M

pytestmark = pytest.mark.gpu

SHIFT = 1e-6          # about eight roundings of an entry of order one in fp32
BLOCKS = 40


def block(n, indefinite, rng):
    r = n // 8
    f = rng.standard_normal((n, r))
    sign = np.where(rng.random(r) < 0.5, -1.0, 1.0) if indefinite else np.ones(r)
    a = (f * sign) @ f.T / r + SHIFT * np.eye(n)
    return ((a + a.T) / 2).astype(np.float32)


def fma(a, b, c):
    """a b + c in fp32, rounded once (the product of two fp32 numbers is exact in fp64; the sum all but)."""
    return (a.astype(np.float64) * np.asarray(b, np.float64) + c).astype(np.float32)


def term_by_term(a):
    """log|det| by steps of pivoting over the whole of the block in fp32, every sum in the order of its terms."""
    n, diag, left = len(a), np.diag(a).copy(), np.ones(len(a), bool)
    low, d, total = np.zeros((n, n), np.float32), np.zeros(n, np.float32), 0.0
    for j in range(n):
        p = int(np.argmax(np.where(left, np.abs(diag), -1)))
        v, w = a[p].copy(), low[p, :j] * d[:j]
        for k in range(j):
            v = fma(-low[:, k], w[k], v)
        d[j], left[p] = diag[p], False
        total += float(np.log(abs(np.float64(d[j]))))
        low[:, j] = np.where(left, v / d[j], np.float32(0))
        diag = fma(-low[:, j], v, diag)
    return total


# A root mean square over 40 blocks scatters by 1 / sqrt(2 * 40), a quotient of two by 16 %: 1.5 is three times that
# above one.  The leaf's matrix is reduced after every 16 steps, both triangles by themselves, which rounds an entry
# and its mirror image apart: a factor of two.
@pytest.mark.parametrize("indefinite", [False, True])
@pytest.mark.parametrize("n, b, flags, bound", [(64, 64, M.FLAG_PIVOT_BLOCK, 1.5), (128, 128, M.FLAG_PIVOT_BLOCK, 1.5),
                                                (64, 64, M.FLAG_PIVOT, 2.0)])
def test_error_is_that_of_sums_term_by_term(n, b, flags, bound, indefinite):
    rng = np.random.default_rng(n + indefinite)
    here, model = [], []
    for _ in range(BLOCKS):
        a = block(n, indefinite, rng)
        want = np.linalg.slogdet(a.astype(np.float64))[1]
        got = M.mdet_logdet_device(torch.from_numpy(a).cuda(), block_size=b, flags=flags)
        assert got.status == 0
        here.append(got.logabsdet - want)
        model.append(term_by_term(a) - want)
    rms = [float(np.sqrt(np.mean(np.square(e)))) for e in (here, model)]
    assert rms[0] <= bound * rms[1], rms
