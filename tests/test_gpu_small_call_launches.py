"""Calls of few launches: pivots that go out with the results at orders around whole workgroups of that launch
(1024 entries), the status words reset by the launch that copies the matrix (a call behind one that
failed), and general matrices at the orders where row tasks of two columns begin (four pairs of tile rows)
against block columns, whose bits they share.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def spd(n, dtype):
    g = torch.Generator().manual_seed(n)
    a = torch.rand((n, n), generator=g, dtype=torch.float64) / n
    a = a + a.T
    a.diagonal().add_(1 + torch.rand(n, generator=g, dtype=torch.float64))
    return a.to("cuda", dtype)


def whole_pieces(a):
    """A copy that is factored in place: rows of a multiple of four elements."""
    n = a.shape[0]
    return torch.zeros((n, (n + 3) // 4 * 4), dtype=a.dtype, device="cuda")[:, :n].copy_(a)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 2049])
def test_pivots_come_out_whole(n, dtype):
    import paper_2503_04424_amd as M
    M.load()
    a = spd(n, dtype)
    diag = torch.full((n + 8,), 7.0, dtype=dtype, device="cuda")
    r = M.mdet_logdet_device(a, diag=diag[:n])
    w = whole_pieces(a)
    inplace = M.mdet_logdet_device(w, overwrite=True)
    assert r.status == 0 and r.logabsdet == inplace.logabsdet
    assert torch.equal(diag[:n], w.diagonal()) and bool((diag[n:] == 7.0).all())


@pytest.mark.parametrize("wide", [False, True])
def test_a_call_behind_one_that_failed(wide):
    import paper_2503_04424_amd as M
    M.load()
    flags = M.FLAG_COMPUTE_F64 if wide else 0
    a = spd(300, torch.float32)
    want = M.mdet_logdet_device(a, flags=flags)
    bad = a.clone()
    bad[200, 200] = float("nan")
    r = M.mdet_logdet_device(bad, flags=flags, raise_on_error=False)
    assert r.status != 0 and r.bad_pivot_index == 200
    again = M.mdet_logdet_device(a, flags=flags)
    assert again.status == 0 and again.bad_pivot_index == -1 and again.logabsdet == want.logabsdet


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [448, 512, 513, 577, 640, 705, 1100])
def test_general_orders_around_four_pairs_of_tile_rows(n, dtype):
    import paper_2503_04424_amd as M
    M.load()
    g = torch.Generator().manual_seed(n)
    a = torch.randn((n, n), generator=g, dtype=torch.float64) / n ** 0.5
    a.diagonal().add_(3.0)
    a = a[torch.argsort(torch.rand(n, generator=g) + torch.arange(n) // 64)].to("cuda", dtype)
    got = []
    for flags in (M.FLAG_GENERAL, M.FLAG_GENERAL | M.FLAG_PROFILE):        # (a profile is of block columns)
        w = whole_pieces(a)
        diag = torch.empty(n, dtype=dtype, device="cuda")
        perm = torch.empty(n, dtype=torch.int32, device="cuda")
        r = M.mdet_logdet_device(w, block_size=128, overwrite=True, flags=flags, diag=diag, perm=perm)
        got.append((diag.cpu(), perm.cpu(), w.cpu(), r.logabsdet, r.sign))
    assert all(torch.equal(x, y) for x, y in zip(got[0][:3], got[1][:3])) and got[0][3:] == got[1][3:]
    assert np.array_equal(np.sort(got[0][1].numpy()), np.arange(n))
