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
