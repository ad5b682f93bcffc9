"""Pivoting over the whole diagonal block where the pivots are not the rows that a group of 64 steps holds in
LDS, those of the largest diagonal entries as it begins: rows in pairs, of which the second all but
vanishes when the first is taken.  Against an elimination in numpy.

Pairs 2 % apart and residuals of 1 - 0.999^2 = 0.002 of the diagonal keep the order determined; a
residual carries the roundings of a few sums of the diagonal's size, 500 units a rounding.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def paired(n, bs, t):
    a = np.zeros((n, n))
    for k in range(0, n, bs):
        w = min(bs, n - k)
        half = w // 2
        rows = k + np.random.default_rng(w).permutation(w)
        d = 1.02 ** -np.arange(w - half) * (-1.0) ** np.arange(w - half)
        for q in range(w - half):
            i = rows[q]
            a[i, i] = d[q]
            if q < half:
                j = rows[w - 1 - q]
                a[j, j] = d[q] * 0.9999
                a[i, j] = a[j, i] = 0.999 * d[q]
    return a.astype(t)


def eliminate(a, bs):
    n, diag, order = a.shape[0], [], []
    for k in range(0, n, bs):
        s = a[k:k + bs, k:k + bs].astype(np.float64)           # (blocks are not coupled)
        left = np.ones(len(s), bool)
        for _ in range(len(s)):
            p = int(np.argmax(np.where(left, np.abs(np.diagonal(s)), -1.0)))
            left[p] = False
            diag.append(s[p, p])
            order.append(k + p)
            l = np.where(left, s[:, p] / s[p, p], 0.0)
            s -= np.outer(l, s[p])
    return np.array(diag), np.array(order)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs", [(66, 128), (128, 128), (256, 256), (300, 320), (512, 512), (700, 256)])
def test_pivots_that_are_not_held(n, bs, dtype):
    import paper_2503_04424_amd as M
    M.load()
    t = np.float64 if dtype == "f64" else np.float32
    a = paired(n, bs, t)
    want, order = eliminate(a, bs)
    guess = np.argsort(-np.abs(np.diagonal(a)[:min(n, bs)]), kind="stable")[:64]
    assert len(set(guess) - set(order[:64])) > 0               # some that are held are not taken in this group
    ad = torch.from_numpy(a).cuda()
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=bs, flags=M.FLAG_PIVOT_BLOCK, diag=diag, perm=perm)
    assert np.array_equal(perm.cpu().numpy(), order)
    assert np.all(np.abs(diag.cpu().numpy().astype(np.float64) - want) <= 4000 * np.finfo(t).eps * np.abs(want))
    assert r.status == 0 and r.sign == int(np.prod(np.sign(want)))
