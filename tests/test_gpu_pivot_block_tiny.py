"""Pivoting over the whole diagonal block with pivots whose reciprocal overflows (subnormal
numbers of the last binades): the quotient of a step is a division there, in every kernel of the
elimination, so that such a pivot is an ordinary one.  All values are exact: powers of two, or
halves and three halves of them.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# per type: a subnormal power of two whose reciprocal is infinite
TINY = {"f64": (np.float64, 2.0 ** -1060), "f32": (np.float32, 2.0 ** -140)}


def run(a, bs):
    import paper_2503_04424_amd as M
    M.load()
    ad = torch.from_numpy(a).cuda()
    n = a.shape[0]
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=bs, flags=M.FLAG_PIVOT_BLOCK, diag=diag, perm=perm, raise_on_error=False)
    return r, diag.cpu().numpy().astype(np.float64), perm.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs", [(3, 64), (20, 64), (256, 256), (300, 320), (600, 640)])
def test_two_tiny_pivots_that_are_not_coupled(n, bs, dtype):
    t, tiny = TINY[dtype]
    d = np.ones(n)
    d[1], d[n - 1] = -2 * tiny, tiny
    r, diag, perm = run(np.diag(d).astype(t), bs)
    order = [i for i in range(n) if i not in (1, n - 1)] + [1, n - 1]
    assert r.status == 0 and r.sign == -1 and r.negative_pivots == 1
    assert np.array_equal(perm, order) and np.array_equal(diag, d[order])
    assert abs(r.logabsdet - 2 * np.log(2.0 * tiny) + np.log(2.0)) <= 1e-12 * abs(r.logabsdet)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_a_tiny_pivot_and_a_row_coupled_to_it(dtype):
    t, tiny = TINY[dtype]
    a = np.eye(20)
    a[4, 4] = a[9, 9] = 4 * tiny
    a[4, 9] = a[9, 4] = 2 * tiny
    r, diag, perm = run(a.astype(t), 64)
    assert r.status == 0 and r.sign == 1
    assert list(perm[-2:]) == [4, 9] and list(diag[-2:]) == [4 * tiny, 3 * tiny]


# Pivots at the other end of the range, where the reciprocal is subnormal, and on both sides of the line from which on a
# step scales them down (2^1021, fp32 2^125).
HUGE = {"f64": (np.float64, (1023, 1021, 1020, 1019)), "f32": (np.float32, (127, 125, 124, 123))}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs", [(20, 64), (300, 320), (600, 640)])
@pytest.mark.parametrize("k", range(4))
def test_a_huge_pivot_and_rows_coupled_to_it(n, bs, dtype, k):
    import paper_2503_04424_amd as M
    M.load()
    t, exponents = HUGE[dtype]
    d = 2.0 ** exponents[k]
    a = np.eye(n)
    a[7, 7], a[3, 3] = d, d / 2
    a[7, 3] = a[3, 7] = 0.75 * d                  # l = 3/4, and d / 2 - 9/16 d is left
    a[7, 5] = a[5, 7] = 2.0 ** (exponents[k] // 2)    # l = 2^(e / 2 - e), and one less 2^(2 (e / 2) - e)
    ad = torch.from_numpy(a.astype(t)).cuda()
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=bs, flags=M.FLAG_PIVOT_BLOCK, diag=diag, perm=perm, overwrite=True,
                             raise_on_error=False)
    assert r.status == 0
    perm, diag, low = list(perm.cpu().numpy()), diag.cpu().numpy().astype(np.float64), ad.cpu().numpy().astype(np.float64)
    assert perm[:2] == [7, 3] and list(diag[:2]) == [d, -0.0625 * d]
    assert low[1, 0] == 0.75 and low[perm.index(5), 0] == 2.0 ** (exponents[k] // 2) / d
