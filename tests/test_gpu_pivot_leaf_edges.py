"""Leaves with pivoting of every awkward width, against oracle.ldlt_pivoted: row order, pivots, sign
and the returned factor, on matrices with a determined order whose pivots move by a hundred
tolerances and more (separated.py); and candidates that differ in the last bits of their fraction
only.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import separated

pytestmark = pytest.mark.gpu


def run(a):
    import paper_2503_04424_amd as M
    M.load()
    n = a.shape[0]
    ad = separated.device_matrix(a)
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=128, flags=M.FLAG_PIVOT, diag=diag, perm=perm, overwrite=True)
    return r, diag.cpu().numpy().astype(np.float64), perm.cpu().numpy(), ad.cpu().numpy().astype(np.float64)


def compare(n, dtype):
    a = separated.matrix(n, dtype)
    o = separated.expected(a, 64, dtype)
    separated.check(o, 64, dtype, *run(a))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 127, 129])
def test_leaf_of_any_width(n, dtype):
    compare(n, dtype)


def test_candidates_that_differ_in_the_last_bits():
    n = 64
    a = np.diag(1.0 + np.arange(n) * 2.0 ** -50)         # the last one is the largest
    a[17, 17] = a[40, 40] = -(1.0 + 100 * 2.0 ** -50)     # but for these two, equal in magnitude
    o = oracle.ldlt_pivoted(a)
    r, d, p, _ = run(a)
    assert list(o.perm[:3]) == [17, 40, 63] and np.array_equal(p, np.asarray(o.perm))
    assert r.sign == o.sign == 1 and np.array_equal(d, np.asarray(o.diag, dtype=np.float64))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [130, 143, 191, 192, 193, 300, 513])
def test_pairs_of_leaves_with_rows_below(n, dtype):
    """The first leaf's order is undone while its rows are read: rows of every remainder, as above."""
    compare(n, dtype)
