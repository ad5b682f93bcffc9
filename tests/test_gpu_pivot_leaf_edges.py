"""Leaves with pivoting of every awkward width, against oracle.ldlt_pivoted: row order, pivots, sign;
and candidates that differ in the last bits of their fraction only.

Separated candidates (magnitudes 3 + 0.01 i in random order, off-diagonal entries of size
1/(4 n)): the eliminated terms move a candidate by less than 0.005 in all, so the order is
determined.  Pivots to 1e-12 (fp32: 1e-5): at most 129 products of size <= 1e-1, rounded once.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


def run(a):
    import paper_2503_04424_amd as M
    M.load()
    n = a.shape[0]
    ad = torch.from_numpy(a).cuda()
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=128, flags=M.FLAG_PIVOT, diag=diag, perm=perm)
    return r, diag.cpu().numpy().astype(np.float64), perm.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 127, 129])
def test_leaf_of_any_width(n, dtype):
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (8 * n)
    a = a + a.T
    np.fill_diagonal(a, (3 + 0.01 * rng.permutation(n)) * rng.choice([-1, 1], n))
    a = a.astype(np.float64 if dtype == "f64" else np.float32)
    o = oracle.ldlt_pivoted(a)
    r, d, p = run(a)
    assert r.status == 0 and r.sign == o.sign and r.negative_pivots == o.negative_pivots
    assert np.array_equal(p, np.asarray(o.perm))
    assert np.max(np.abs(d - o.diag) / np.abs(o.diag)) < (1e-12 if dtype == "f64" else 1e-5)


def test_candidates_that_differ_in_the_last_bits():
    n = 64
    a = np.diag(1.0 + np.arange(n) * 2.0 ** -50)         # the last one is the largest
    a[17, 17] = a[40, 40] = -(1.0 + 100 * 2.0 ** -50)     # but for these two, equal in magnitude
    o = oracle.ldlt_pivoted(a)
    r, d, p = run(a)
    assert list(o.perm[:3]) == [17, 40, 63] and np.array_equal(p, np.asarray(o.perm))
    assert r.sign == o.sign == 1 and np.array_equal(d, np.asarray(o.diag, dtype=np.float64))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [130, 143, 191, 192, 193, 300, 513])
def test_pairs_of_leaves_with_rows_below(n, dtype):
    """The first leaf's order is undone while its rows are read: rows of every remainder, as above."""
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (8 * n)
    a = a + a.T
    np.fill_diagonal(a, (3 + 0.01 * rng.permutation(n)) * rng.choice([-1, 1], n))
    a = a.astype(np.float64 if dtype == "f64" else np.float32)
    o = oracle.ldlt_pivoted(a)
    r, d, p = run(a)
    assert r.status == 0 and r.sign == o.sign and r.negative_pivots == o.negative_pivots
    assert np.array_equal(p, np.asarray(o.perm))
    # an off-diagonal entry of the wrong column changes a pivot by about 1 / (4 n)^2 / 3 > 8e-8;
    # fp32 rounds the pivot itself by 6e-8 relative, so only fp64 can show it
    assert np.max(np.abs(d - o.diag) / np.abs(o.diag)) < (1e-12 if dtype == "f64" else 1e-5)
