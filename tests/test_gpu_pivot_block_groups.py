"""Pivoting over the whole diagonal block at the sizes where its elimination changes kernels (one
workgroup of 256 or 512 threads per group of 64 steps, or a launch per step) and where the
block or the last group is ragged, against oracle.ldlt_pivoted.

Matrices with a determined order whose pivots move by a hundred tolerances and more (separated.py);
permutation, pivots and the returned factor, so that a wrong multiplier shows at first order.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import separated

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs", [(1, 64), (15, 64), (17, 64), (64, 64), (65, 128), (255, 256), (256, 256),
                                  (257, 320), (300, 128), (511, 512), (512, 512), (513, 576), (640, 512)])
def test_every_kernel_takes_the_oracles_order(n, bs, dtype):
    import paper_2503_04424_amd as M
    M.load()
    a = separated.matrix(n, dtype)
    o = separated.expected(a, bs, dtype)
    ad = separated.device_matrix(a)
    diag = torch.empty(n, dtype=ad.dtype, device="cuda")
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    r = M.mdet_logdet_device(ad, block_size=bs, flags=M.FLAG_PIVOT_BLOCK, diag=diag, perm=perm, overwrite=True)
    separated.check(o, bs, dtype, r, diag.cpu().numpy().astype(np.float64), perm.cpu().numpy(),
                    ad.cpu().numpy().astype(np.float64))
