"""Leaves whose width is not a multiple of the 16-column sub-blocks they are factored in, alone
and with rows below them, through the step entry point (its chain of launches; whole calls:
test_gpu_flow.py), against the oracle's factor.

Tolerance: the pivots of these matrices (diagonal 1 .. 4, off-diagonal entries of size
1/(2 w)) are sums of at most 64 products of size <= 1; a double-precision elimination in any
order is within a few hundred units in the last place, 1e-13 (fp32: 1e-5).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e12, 1e-12])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("w", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
def test_leaf_of_any_width(w, dtype, scale):
    import paper_2503_04424_amd as M
    M.load()
    npdt, tol = (np.float64, 1e-13) if dtype == "f64" else (np.float32, 1e-5)
    for below in (0, 1, 70):
        m = w + below
        rng = np.random.default_rng(100 * w + below)
        a = rng.uniform(-1, 1, (m, m)) / (2 * w)
        a = a + a.T
        np.fill_diagonal(a, rng.uniform(1, 4, m) * rng.choice([-1, 1], m))
        a = (a * scale).astype(npdt)
        # the oracle on the leading w columns: eliminate them, rows below included
        ref = a.astype(np.longdouble)
        piv = np.zeros(w, np.longdouble)
        for j in range(w):
            piv[j] = ref[j, j]
            l = ref[j + 1:, j] / piv[j]
            ref[j + 1:, j + 1:] -= np.outer(l, ref[j, j + 1:])
            ref[j + 1:, j] = l
        if below == 0:
            o = oracle.ldlt_logdet(a, want_diag=True)
            assert np.max(np.abs(o.diag - piv) / np.abs(piv)) < 1e-13
        ld = (m + 3) // 4 * 4
        buf = torch.zeros((m, ld), dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda")
        buf[:, :m] = torch.from_numpy(a).cuda()
        upper = torch.triu(buf[:, :m], 1).cpu()
        d = torch.zeros(w, dtype=buf.dtype, device="cuda")
        dinv = torch.zeros_like(d)
        flags = torch.full((2 + 1024,), -1, dtype=torch.int64, device="cuda")
        M.mdet_step_panel_factor(buf[:, :m], w, d, dinv, flags)
        torch.cuda.synchronize()
        got = buf[:, :m].cpu().numpy().astype(np.longdouble)
        assert np.max(np.abs(d.cpu().numpy() - piv) / np.abs(piv)) < tol
        assert np.max(np.abs(dinv.cpu().numpy().astype(np.longdouble) * piv - 1)) < tol
        i, j = np.indices((m, w))
        low = i > j
        if low.any():
            assert np.max(np.abs(got[:, :w] - ref[:, :w])[low]) < tol
        # what lies above the diagonal, and right of the leaf, is left alone
        assert torch.equal(torch.triu(buf[:, :m], 1).cpu()[:, :w], upper[:, :w])
        assert int(flags[0].item()) == -1
