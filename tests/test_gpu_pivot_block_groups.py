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


@pytest.mark.parametrize("n,bs,dtype", [(192, 64, "f64"), (300, 128, "f32"), (448, 192, "f64"), (449, 192, "f32"),
                                        (300, 256, "f64"), (6400, 192, "f64"), (3711, 640, "f64"), (3712, 640, "f64"),
                                        (6144 + 576, 576, "f32")])
def test_rows_below_on_either_stream_give_the_same_bits(n, bs, dtype):
    """Block columns on both sides of the rule that puts the rows below a diagonal block on a stream of their own
    (how many groups of steps, how many rows), and both kinds in one call, against one stream only."""
    import paper_2503_04424_amd as M
    M.load()
    td = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator().manual_seed(n)
    a = torch.rand((n, n), generator=g, dtype=torch.float32).to("cuda", td) / n
    a = torch.tril(a) + torch.tril(a, -1).T
    a.diagonal().copy_((torch.rand(n, generator=g) * 3 + 1) * (torch.randint(0, 2, (n,), generator=g) * 2 - 1))
    got = []
    for flags in (M.FLAG_PIVOT_BLOCK, M.FLAG_PIVOT_BLOCK | M.FLAG_NO_LOOKAHEAD):
        w = torch.zeros((n, (n + 3) // 4 * 4), dtype=td, device="cuda")[:, :n].copy_(a)
        diag = torch.empty(n, dtype=td, device="cuda")
        perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        r = M.mdet_logdet_device(w, block_size=bs, flags=flags, diag=diag, perm=perm, overwrite=True)
        assert r.status == 0
        got.append((diag.cpu(), perm.cpu(), torch.tril(w).cpu(), r.logabsdet, r.sign))
    assert not torch.equal(got[0][1], torch.arange(n, dtype=torch.int32))
    assert torch.equal(torch.sort(got[0][1])[0], torch.arange(n, dtype=torch.int32))
    assert all(torch.equal(x, y) for x, y in zip(got[0][:3], got[1][:3])) and got[0][3:] == got[1][3:]
