"""Block columns factored by one launch (panel_flow_kernel): orders around the edges of tiles and pairs
of tiles, rows that do not start on 128-byte lines, several launches, the scaled copy.

Tolerance: diagonal 1 .. 4 with either sign (positive for the Cholesky form), off-diagonal entries of
size 1 / (2 n): every entry of the factor is a sum of at most n products of size <= 1 / n, so an
elimination in any order is within a few hundred units in the last place, 1e-13 (fp32: 1e-5).
Whatever the block columns, the products of an entry are summed in one order: same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["sym", "spd"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [65, 127, 128, 129, 191, 193, 256, 321, 448, 640, 1025])
def test_orders_around_tile_edges(n, dtype, form):
    import paper_2503_04424_amd as M
    M.load()
    npdt, tol = (np.float64, 1e-13) if dtype == "f64" else (np.float32, 1e-5)
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (2 * n)
    a = a + a.T
    np.fill_diagonal(a, rng.uniform(1, 4, n) * (rng.choice([-1, 1], n) if form == "sym" else 1))
    a = a.astype(npdt)
    o = oracle.ldlt_logdet(a.astype(np.float64), want_diag=True)
    flags = M.FLAG_ASSUME_SPD if form == "spd" else 0
    got = []
    # whole lines and rows that straddle them, one launch and several, look-ahead and one stream
    vec = 16 // np.dtype(npdt).itemsize
    lds = [(n + 31) // 32 * 32, (n + vec - 1) // vec * vec, (n + 31) // 32 * 32 + vec]
    for ld, bs, extra in [(lds[0], 1024, 0), (lds[1], 128, 0), (lds[2], 64, 0), (lds[0], 64, M.FLAG_NO_LOOKAHEAD),
                          (lds[1], 192, M.FLAG_PROFILE), (lds[2], 128, 0 if form == "spd" else M.FLAG_SCALED_COPY)]:
        buf = torch.full((n, ld), float("nan"), dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda")
        buf[:, :n] = torch.from_numpy(np.tril(a)).cuda()
        buf[:, :n] += torch.triu(torch.full((n, n), float("nan"), dtype=buf.dtype, device="cuda"), 1)
        diag = torch.empty(n, dtype=buf.dtype, device="cuda")
        r = M.mdet_logdet_device(buf[:, :n], block_size=bs, overwrite=True, flags=flags | extra, diag=diag)
        d = diag.cpu().numpy().astype(np.float64)
        assert r.status == 0 and np.max(np.abs(d - o.diag) / np.abs(o.diag)) < tol, (ld, bs)
        assert r.flops == pytest.approx(2 * (n ** 3 - n) / 6, rel=1e-12)
        f = buf[:, :n].cpu().numpy()
        assert np.isnan(f[np.triu_indices(n, 1)]).all()              # what lies above the diagonal is not used
        got.append((d, np.tril(f)))
    for d, f in got[1:]:
        assert np.array_equal(d, got[0][0]) and np.array_equal(f, got[0][1])
    # the factor itself, against the matrix
    low = np.tril(got[0][1].astype(np.float64), -1)
    if form == "spd":                                                # stored leaves are unit-lower, rows below them L D^(1/2)
        for k in range(0, n, 64):
            low[k + 64:, k:k + 64] /= np.sqrt(got[0][0][k:k + 64])
    low += np.eye(n)
    err = np.abs(low * got[0][0] @ low.T - a.astype(np.float64))
    assert err.max() < 8 * tol                                       # entries up to 4


@pytest.mark.parametrize("form", ["sym", "spd"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("w", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
def test_leaf_of_any_width_in_a_whole_call(w, dtype, form):
    """The last leaf of a call, alone and behind whole ones, at three scales (the step entry point's leaf:
    test_gpu_leaf_edges.py)."""
    import paper_2503_04424_amd as M
    M.load()
    npdt, tol = (np.float64, 1e-13) if dtype == "f64" else (np.float32, 1e-5)
    for n, scale in [(w, 1.0), (w, 1e12), (w, 1e-12), (64 + w, 1.0), (128 + w, 1.0)]:
        rng = np.random.default_rng(100 * n + w)
        a = rng.uniform(-1, 1, (n, n)) / (2 * n)
        a = a + a.T
        np.fill_diagonal(a, rng.uniform(1, 4, n) * (rng.choice([-1, 1], n) if form == "sym" else 1))
        a = (a * scale).astype(npdt)
        o = oracle.ldlt_logdet(a.astype(np.float64), want_diag=True)
        diag = torch.empty(n, dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda")
        r = M.mdet_logdet_device(torch.from_numpy(a).cuda(), flags=M.FLAG_ASSUME_SPD if form == "spd" else 0, diag=diag)
        d = diag.cpu().numpy().astype(np.float64)
        assert r.status == 0 and r.sign == o.sign and np.max(np.abs(d - o.diag) / np.abs(o.diag)) < tol, (n, scale)


@pytest.mark.parametrize("form", ["gen", "pivot"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [64, 65, 128, 129, 193, 320, 449, 1025])
def test_pivoting_forms_around_tile_edges(n, dtype, form):
    """Pivots that stand in the first place of no leaf: the largest of each leaf's columns (diagonals) is in
    its last rows.  The factor multiplied out gives the matrix, and the block columns change no bit."""
    import paper_2503_04424_amd as M
    M.load()
    npdt, tol = (np.float64, 1e-13) if dtype == "f64" else (np.float32, 1e-5)
    rng = np.random.default_rng(n + 1)
    a = rng.uniform(-1, 1, (n, n)) / (2 * n)
    if form == "pivot":
        a = a + a.T
        np.fill_diagonal(a, (1 + np.arange(n) % 64 / 21.0) * rng.choice([-1, 1], n))     # 1 .. 4, the last the largest
    else:
        np.fill_diagonal(a, rng.uniform(1, 4, n))
        rows = np.arange(n)
        for k in range(0, n, 64):
            rows[k:k + 64] = rows[k:k + 64][::-1]
        a = a[rows]
    a = a.astype(npdt)
    vec = 16 // np.dtype(npdt).itemsize
    got = []
    for ld, bs, extra in [((n + 31) // 32 * 32, 1024, 0), ((n + vec - 1) // vec * vec, 128, 0),
                          ((n + 31) // 32 * 32 + vec, 64, 0), ((n + 31) // 32 * 32, 192, M.FLAG_PROFILE)]:
        buf = torch.zeros((n, ld), dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda")
        buf[:, :n] = torch.from_numpy(a).cuda()
        diag = torch.empty(n, dtype=buf.dtype, device="cuda")
        perm = torch.empty(n, dtype=torch.int32, device="cuda")
        r = M.mdet_logdet_device(buf[:, :n], block_size=bs, overwrite=True, diag=diag, perm=perm,
                                 flags=extra | (M.FLAG_GENERAL if form == "gen" else M.FLAG_PIVOT))
        assert r.status == 0 and r.flops == pytest.approx((4 if form == "gen" else 2) * (n ** 3 - n) / 6, rel=1e-12)
        got.append((diag.cpu().numpy(), perm.cpu().numpy(), buf[:, :n].cpu().numpy()))
    for d, p, f in got[1:]:
        assert np.array_equal(d, got[0][0]) and np.array_equal(p, got[0][1])
        assert np.array_equal(*(f_ if form == "gen" else np.tril(f_) for f_ in (f, got[0][2])))
    d, p, f = got[0][0].astype(np.float64), got[0][1], got[0][2].astype(np.float64)
    assert not np.array_equal(p[:64], np.arange(min(n, 64)))
    if form == "gen":
        want = np.linalg.slogdet(a.astype(np.float64))
        assert r.sign == want[0] and abs(r.logabsdet - want[1]) <= 10 * n * tol
    # rows of a later leaf stay in their input order in the columns of the leaves before it
    low = np.tril(f, -1)
    up = np.triu(f, 1) if form == "gen" else low.T
    exact = a.astype(np.float64)
    s = exact.copy()
    for k in range(0, n, 64):
        e = min(n, k + 64)
        q = p[k:e]
        l11, u11 = low[k:e, k:e] + np.eye(e - k), up[k:e, k:e] + np.eye(e - k)
        lead = s[k:e, k:e][q - k] if form == "gen" else s[k:e, k:e][np.ix_(q - k, q - k)]
        assert np.abs(l11 * d[k:e] @ u11 - lead).max() < 8 * tol
        l21, u12 = low[e:, k:e], up[k:e, e:]
        cols = s[e:, k:e] if form == "gen" else s[e:, k:e][:, q - k]
        assert e == n or np.abs(l21 * d[k:e] @ u11 - cols).max() < 8 * tol
        right = s[k:e, e:][q - k]
        assert e == n or np.abs(l11 * d[k:e] @ u12 - right).max() < 8 * tol
        s[e:, e:] -= l21 * d[k:e] @ u12


@pytest.mark.parametrize("form", ["sym", "gen"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [129, 323])
def test_copy_without_room_for_long_rows(n, dtype, form):
    """The least budget that the plan accepts, and a workspace of that size, leave no room for rows of the copy
    on 128-byte lines: same bits by the route that reads past the caches."""
    import paper_2503_04424_amd as M
    M.load()
    flags = M.FLAG_GENERAL if form == "gen" else 0
    roomy = M.mdet_workspace_query(n, dtype, 64, 0, False, flags, True)[0]
    low, high = 0, roomy
    while high - low > 1:
        mid = (low + high) // 2
        try:
            M.mdet_workspace_query(n, dtype, 64, mid, False, flags, True)
            high = mid
        except M.MemdetError:
            low = mid
    assert high < roomy
    td = torch.float64 if dtype == "f64" else torch.float32
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (2 * n)
    a = a + a.T + np.diag(rng.uniform(1, 4, n))
    a = torch.from_numpy(a).to(td).cuda()
    own = torch.empty(high, dtype=torch.uint8, device="cuda")
    got = []
    for kw in ({}, {"mem_budget": high}, {"workspace": own}):
        diag = torch.empty(n, dtype=td, device="cuda")
        r = M.mdet_logdet_device(a, block_size=64, flags=flags, diag=diag, **kw)
        assert r.status == 0
        got.append((diag.cpu().numpy(), r.logabsdet, r.sign))
    for d, v, s in got[1:]:
        assert np.array_equal(d, got[0][0]) and (v, s) == got[0][1:]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 3, 63, 65, 130, 131, 257])
def test_copy_of_a_view_of_some_columns(n, dtype):
    """Rows longer than the order, copied in pieces of 16 bytes and, where they are not whole ones, by entry: the
    same bits as from rows without a gap, and nothing between the rows is touched or used."""
    import paper_2503_04424_amd as M
    M.load()
    td, vec = (torch.float64, 2) if dtype == "f64" else (torch.float32, 4)
    rng = np.random.default_rng(n)
    a = rng.uniform(-1, 1, (n, n)) / (2 * n)
    a = torch.from_numpy(a + a.T + np.diag(rng.uniform(1, 4, n))).to(td).cuda()
    got = []
    for ld in (n, (n + vec - 1) // vec * vec, (n + vec - 1) // vec * vec + vec):
        flat = torch.full(((n - 1) * ld + n,), float("nan"), dtype=td, device="cuda")
        view = flat.as_strided((n, n), (ld, 1))
        view.copy_(a)
        before = flat.clone()
        diag = torch.empty(n, dtype=td, device="cuda")
        r = M.mdet_logdet_device(view, block_size=64, diag=diag)
        assert r.status == 0 and torch.equal(flat.isnan(), before.isnan()) and torch.equal(view, a)
        got.append((diag.cpu().numpy(), r.logabsdet))
    for d, v in got[1:]:
        assert np.array_equal(d, got[0][0]) and v == got[0][1]


@pytest.mark.parametrize("n", [1, 64, 1023, 1024, 1025, 1040])
@pytest.mark.parametrize("bs", [64, 128])
def test_results_of_few_and_many_blocks(n, bs):
    """The sums of log|d| over block columns, by the one launch of up to 16 of them and by the two of more:
    a diagonal matrix, whose pivots are exact and one of which is not positive."""
    import paper_2503_04424_amd as M
    M.load()
    d = np.random.default_rng(n).uniform(0.5, 4, n)
    d[n // 2] *= -1
    r = M.mdet_logdet_device(torch.from_numpy(np.diag(d)).cuda(), block_size=bs)
    want = float(np.sum(np.log(np.abs(d).astype(np.longdouble))))
    assert (r.status, r.sign, r.negative_pivots) == (0, -1, 1) and abs(r.logabsdet - want) <= 4e-16 * n


def multiplied_out(form, a, d, p, f):
    """Largest difference between the matrix and the factor multiplied out (all fp64, on the GPU); rows of a leaf
    stand in their input order in the columns of the leaves before it."""
    n = a.shape[0]
    low = torch.tril(f, -1)
    if form in ("sym", "spd"):
        if form == "spd":                                # stored leaves are unit-lower, rows below them L D^(1/2)
            for k in range(0, n, 64):
                low[k + 64:, k:k + 64] /= torch.sqrt(d[k:k + 64])
        low += torch.eye(n, dtype=f.dtype, device=f.device)
        return float(torch.abs((low * d) @ low.T.contiguous() - a).max())
    up = torch.triu(f, 1) if form == "gen" else low.T.contiguous()
    s, worst = a.clone(), 0.0
    for k in range(0, n, 64):
        e = min(n, k + 64)
        q = p[k:e].long() - k
        eye = torch.eye(e - k, dtype=f.dtype, device=f.device)
        l11, u11 = low[k:e, k:e] + eye, up[k:e, k:e] + eye
        lead = s[k:e, k:e][q] if form == "gen" else s[k:e, k:e][q][:, q]
        diffs = [(l11 * d[k:e]) @ u11 - lead]
        if e < n:
            l21, u12 = low[e:, k:e].contiguous(), up[k:e, e:].contiguous()
            cols = s[e:, k:e] if form == "gen" else s[e:, k:e][:, q]
            diffs += [(l21 * d[k:e]) @ u11 - cols, (l11 * d[k:e]) @ u12 - s[k:e, e:][q]]
            s[e:, e:] -= (l21 * d[k:e]) @ u12
        worst = max([worst] + [float(torch.abs(x).max()) for x in diffs])
    return worst


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("form,n", [(f, n) for f in ("sym", "spd", "pivot") for n in (3585, 3713, 3776, 3800, 3841)] +
                         [("gen", n) for n in (1793, 1921, 1984, 2049, 2113)])
def test_row_tasks_of_two_columns(form, n, dtype):
    """Orders from which on row tasks take two tile columns (28 pairs of tile rows and one more, general
    matrices 14), with an odd and an even number of tile rows, the last of them whole, ragged or of one row; rows on
    128-byte lines and off them; whole matrices, block columns with and without the scaled copy, and block
    columns of one tile column, which have no such tasks: the same bits, and the factor multiplied out.

    Off-diagonal entries c u with |u| <= 1, c = 1 / (2 sqrt(n)), diagonal 1 .. 4: the terms of an entry add up to
    sum |l| |d| |l| <= n c^2 E u^2 = 1/12 beside the diagonal itself, so an elimination in any order
    leaves |A - L D L^T| <= n u / 12 and a few roundings of numbers up to 5, u the unit roundoff.  64 terms left
    out or taken twice show as 8 c^2 / 3 = 2 / (3 n) on average: ten times that in fp32."""
    import paper_2503_04424_amd as M
    M.load()
    td, unit = (torch.float64, 2.0 ** -53) if dtype == "f64" else (torch.float32, 2.0 ** -24)
    tol = unit * (n / 6 + 64)
    g = torch.Generator().manual_seed(n)
    a = (torch.rand((n, n), generator=g, dtype=torch.float64) * 2 - 1) / (2 * n ** 0.5)
    if form != "gen":
        a = torch.tril(a) + torch.tril(a, -1).T
    big = (1 + torch.arange(n) % 64 / 21.0).double()                 # in every leaf the last the largest
    if form in ("sym", "pivot"):
        big = big * (torch.randint(0, 2, (n,), generator=g) * 2 - 1)
    a.diagonal().copy_(big)
    if form == "gen":
        rows = torch.arange(n)
        for k in range(0, n, 64):
            rows[k:k + 64] = rows[k:k + 64].flip(0)
        a = a[rows]
    a = a.to(td).cuda()
    vec = 16 // a.element_size()
    on, off = (n + 31) // 32 * 32, (n + 31) // 32 * 32 + vec
    flags = {"sym": 0, "spd": M.FLAG_ASSUME_SPD, "pivot": M.FLAG_PIVOT, "gen": M.FLAG_GENERAL}[form]
    scaled = M.FLAG_SCALED_COPY if form in ("sym", "pivot") else 0
    first = None
    for ld, bs, extra in [(on, 4096, 0), (off, 4096, 0), (off, 64, M.FLAG_NO_LOOKAHEAD), (on, 64, 0), (on, 1024, scaled),
                          (off, 640, scaled | M.FLAG_PROFILE), (on, 64, M.FLAG_PROFILE)]:
        w = torch.full((n, ld), float("nan"), dtype=td, device="cuda")[:, :n]
        w.copy_(a)
        diag = torch.empty(n, dtype=td, device="cuda")
        perm = torch.arange(n, dtype=torch.int32, device="cuda")
        r = M.mdet_logdet_device(w, block_size=bs, overwrite=True, flags=flags | extra, diag=diag, perm=perm)
        assert r.status == 0, (ld, bs)
        f = w if form == "gen" else torch.tril(w)
        if first is None:
            first = (diag, perm, f.clone(), r.logabsdet, r.sign)
            if form in ("pivot", "gen"):
                assert not torch.equal(perm[:64].cpu(), torch.arange(64, dtype=torch.int32))
            assert multiplied_out(form, a.double(), diag.double(), perm, f.double()) < tol
        assert all(torch.equal(x, y) for x, y in zip(first[:3], (diag, perm, f))), (ld, bs, extra)
        # (n terms up to 1.4, added in another order: n / 64 + 10 additions at most to each)
        assert abs(r.logabsdet - first[3]) <= 1.4 * n * (n / 64 + 10) * 2.0 ** -53 and r.sign == first[4]
