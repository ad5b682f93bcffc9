"""Leaves of a general matrix of every awkward width, against oracle.lu_logdet: row order, pivots
and sign; and candidates that differ in the last bits of their fraction only.

Gaussian matrices of order <= 64 with the pivot taken among all rows: multipliers are at most
1, so the pivots are good to growth (< 64) times 64 roundings, 1e-12 (fp32: 1e-3); candidates
closer than that do not occur for these seeds.
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
    r = M.mdet_logdet_device(ad, block_size=64, flags=M.FLAG_GENERAL, diag=diag, perm=perm)
    return r, diag.cpu().numpy().astype(np.float64), perm.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 48, 55, 56, 57, 63, 64, 65, 127, 129])
def test_leaf_of_any_width(n, dtype):
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, n))
    if n > 64:                      # more than one group: keep the growth between groups bounded
        a = a / np.sqrt(n) + np.diag(rng.choice([-1, 1], n) * 4.0)[rng.permutation(64).tolist() + list(range(64, n))]
    a = a.astype(np.float64 if dtype == "f64" else np.float32)
    o = oracle.lu_logdet(a)
    r, d, p = run(a)
    assert r.status == 0 and r.sign == o.sign
    assert np.array_equal(p, np.asarray(o.perm))
    assert np.max(np.abs(d - o.diag) / np.abs(o.diag)) < (1e-12 if dtype == "f64" else 1e-3)


def test_candidates_that_differ_in_the_last_bits():
    n = 64
    a = np.eye(n)
    a[:, 0] = 1.0 + np.arange(n)[::-1] * 2.0 ** -50      # the largest on top
    a[17, 0] = 1.0 + 100 * 2.0 ** -50                    # but for this one
    a[40, 0] = 1.0 + 100 * 2.0 ** -50                    # and its equal further down
    o = oracle.lu_logdet(a)
    r, d, p = run(a)
    assert o.perm[0] == 17 and np.array_equal(p, np.asarray(o.perm))
    assert r.sign == o.sign and abs(r.logabsdet - o.logabsdet) < 1e-12
