"""Pivoting over the whole diagonal block at the sizes where its elimination changes kernels (one
workgroup of 256 or 512 threads per group of 64 steps, or a launch per step) and where the
block or the last group is ragged, against oracle.ldlt_pivoted.

Separated candidates (diagonal magnitudes 3 + 0.01 i in random order, off-diagonal entries of
size 1/(4 n)): the eliminated terms move a candidate by at most 1/(16 n) * n / 3 < 0.005 / 2 in
all, so the order is determined and the permutations must be equal.  Pivots to 1e-12 (fp32:
1e-5): at most 640 products of size <= 1e-3 each, rounded once.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs", [(1, 64), (15, 64), (17, 64), (64, 64), (65, 128), (255, 256), (256, 256),
                                  (257, 320), (300, 128), (511, 512), (512, 512), (513, 576), (640, 512)])
def test_every_kernel_takes_the_oracles_order(n, bs, dtype):
    import paper_2503_04424_amd as M
    M.load()
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (8 * n)
    a = a + a.T
    mag = 3 + 0.01 * rng.permutation(n)
    np.fill_diagonal(a, mag * rng.choice([-1, 1], n))
    a = a.astype(np.float64 if dtype == "f64" else np.float32)
    o = oracle.ldlt_pivoted(a, group=bs)
    ad = torch.from_numpy(a).cuda()
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=bs, flags=M.FLAG_PIVOT_BLOCK, diag=diag, perm=perm)
    assert r.status == M.Status.OK and r.sign == o.sign
    assert np.array_equal(perm.cpu().numpy(), np.asarray(o.perm))
    tol = 1e-12 if dtype == "f64" else 1e-5
    assert np.max(np.abs(diag.cpu().numpy().astype(np.float64) - o.diag) / np.abs(o.diag)) < tol
