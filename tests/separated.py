"""Symmetric matrices whose pivoting order is determined and whose pivots and multipliers move by far
more than single precision rounds, whatever their order n; and the comparison of a pivoted
factorisation of one with the oracle's.

a_ij = s_i r_i r_j u_ij c for i != j, a_ii = s_i r_i^2: magnitudes r_i^2 = 3 * 1.03^k in random
order, random signs, 0.7 <= |u| <= 1, c^2 = 0.006 / sqrt(n).  An eliminated pivot k changes
candidate i by a share c^2 u^2 of either sign: at least 0.2 % of some pivot at n = 2, a random walk
of standard deviation 0.45 % over n steps, beside the 3 % between neighbours.  check() asserts
both on the oracle's result: some pivot at least 100 tolerances from the un-eliminated diagonal, none
further than half the distance.  Scaled by r, multipliers are of size c (0.015 at n = 640), a
thousand tolerances, and rounding is that of n <= 640 products of size c^2 added to numbers of
size one: n eps / 2 = 2e-5 at worst in fp32, in random order a tenth of that (an fp32 elimination in
numpy: 2e-6 at n = 640, multipliers 7e-8); 1e-12 in fp64 (n eps = 1.4e-13).
"""
import numpy as np

import oracle

TOL = {"f64": 1e-12, "f32": 1e-5}
NPTYPE = {"f64": np.float64, "f32": np.float32}


def matrix(n, dtype):
    rng = np.random.default_rng(n)
    r = np.sqrt(3 * 1.03 ** rng.permutation(n))
    u = rng.uniform(0.7, 1.0, (n, n)) * rng.choice([-1, 1], (n, n)) * np.sqrt(0.006 / np.sqrt(n))
    u = np.tril(u, -1)
    u = u + u.T + np.diag(rng.choice([-1.0, 1.0], n))
    return (u * r[:, None] * r).astype(NPTYPE[dtype])


def device_matrix(a):
    """On the GPU with a leading dimension that the call works in place on."""
    import torch
    n = a.shape[0]
    ad = torch.zeros((n, (n + 3) // 4 * 4), dtype=torch.from_numpy(a).dtype, device="cuda")[:, :n]
    return ad.copy_(torch.from_numpy(a))


def expected(a, group, dtype):
    n = a.shape[0]
    o = oracle.ldlt_pivoted(a, group=group, want_L=True)
    before = np.diag(a).astype(np.float64)[o.perm]
    moved = np.abs(before - o.diag) / np.abs(o.diag)
    assert o.status == 0 and np.max(moved) < 0.015 and (n == 1 or np.max(moved) > 100 * TOL[dtype])
    return o


def check(o, group, dtype, result, diag, perm, factor):
    """factor: what the call left of the matrix; rows of a group stand in input order in the columns
    before the group."""
    n = len(o.diag)
    assert result.status == 0 and result.sign == o.sign and result.negative_pivots == o.negative_pivots
    assert np.array_equal(perm, o.perm)
    assert np.max(np.abs(diag - o.diag) / np.abs(o.diag)) < TOL[dtype]
    got = factor.copy()
    for g0 in range(group, n, group):
        g1 = min(n, g0 + group)
        got[g0:g1, :g0] = factor[perm[g0:g1], :g0]
    r = np.sqrt(np.abs(o.diag))
    off = np.abs(got - o.L) * r / r[:, None]
    assert np.max(np.tril(off, -1), initial=0.0) < TOL[dtype]
    assert np.max(np.abs(np.diag(got) - o.diag) / np.abs(o.diag)) < TOL[dtype]
