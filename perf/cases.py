"""Performance cases: the work a user of this library has it do, through its public entry points.

`listed()` gives the named cases, `draw(rng)` more of the same ranges.  A case is a dict:

  entry   'memdet' (the front end), 'device' (mdet_logdet_device), 'host' (mdet_logdet_host under
          a device-memory budget), 'sequence' (principal log-determinants and the FLODANCE fit)
  form    'sym' (L D L^T), 'spd' (Cholesky form), 'gen' (P M = L D U), 'pivot' (pivoting inside
          64 columns), 'pivot_block' (pivoting inside a diagonal block)
  store   type the matrix is stored in; `wide`: fp64 arithmetic on a narrower matrix
  kind    what matrix it is (see `matrix`)
  n, b    order and block size (b = 0: the library's choice)
  kept    the caller keeps the workspace between calls, as bench.py does
  factor  the factorisation is done in place and returned
  share   'host': device budget as a share of the packed lower triangle
  q, d    'sequence': correction terms and stride of the fit
"""
import math

import numpy as np
import torch

import paper_2503_04424_amd as M

STORE = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
BYTES = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}
GROUP = 64          # columns among which 'pivot' and 'gen' choose


def _case(name, entry, form, store, kind, n, b=0, wide=False, kept=False, factor=False, share=0.0, q=0, d=0):
    c = dict(entry=entry, form=form, store=store, kind=kind, n=n, b=b, wide=wide, kept=kept, factor=factor,
             share=share, q=q, d=d)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the benchmark's smallest configuration: one log-determinant among many (hyper-parameter search)
        _case("wishart_sym_f64_n512", "device", "sym", "f64", "wishart", 512, 128),
        # a Gaussian-process likelihood on an ordinary, ragged data set, by the front end
        _case("matern_spd_f64_n1500", "memdet", "spd", "f64", "matern32", 1500),
        # the front end's default: a matrix nothing is known of
        _case("general_f64_n2900", "memdet", "gen", "f64", "general", 2900),
        # robust form for indefinite matrices, pivot from the whole diagonal block
        _case("indefinite_pivot_block_f64_n3000", "memdet", "pivot_block", "f64", "indefinite", 3000),
        # its cheaper relative: pivot among 64 columns
        _case("indefinite_pivot_f64_n4096", "memdet", "pivot", "f64", "indefinite", 4096),
        # an NTK Gram matrix kept in 16 bits, log-determinant in 64 (the paper's data-precision pipeline)
        _case("ntk_bf16_wide_spd_n5555", "memdet", "spd", "bf16", "ntk_narrow", 5555, wide=True),
        # the benchmark's n = 8192 configuration, factor wanted too (solves, principal minors)
        _case("se_sym_f64_n8192", "device", "sym", "f64", "se", 8192, 1024, kept=True, factor=True),
        # the benchmark's general-matrix mode at the same order
        _case("general_f64_n8192", "device", "gen", "f64", "general", 8192, 1024, kept=True),
        # fp32 storage and arithmetic on a well-conditioned covariance
        _case("matern_sym_f32_n10000", "memdet", "sym", "f32", "matern32", 10000),
        # larger than its device budget: streamed from ordinary host memory
        _case("host_sym_f64_n12288", "host", "sym", "f64", "matern32", 12288, 1024, kept=True, share=0.45),
        # the benchmark's resident NTK configuration
        _case("ntk_sym_f64_n32768", "device", "sym", "f64", "ntk", 32768, 2048, kept=True),
        # pivots of 50 000 data points with 10 outputs -> scaling-law fit (the paper's experiment size)
        _case("sequence_n500000", "sequence", "sym", "f64", "pivots", 500000, q=4, d=10),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["sym", "spd", "sym", "gen", "pivot", "pivot_block", "wide", "f32", "host", "sequence"])
    entry = rng.choice(["memdet", "device"])
    kept = entry == "device" and rng.random() < 0.5
    if what == "sequence":
        return _case(None, "sequence", "sym", "f64", "pivots", _log_uniform(rng, 5000, 500000), q=rng.randint(0, 6),
                     d=rng.choice([1, 2, 10]))
    if what == "host":
        n = _log_uniform(rng, 3000, 12000)
        return _case(None, "host", "sym", "f64", "matern32", n, max(256, n // 12 // 64 * 64), kept=rng.random() < 0.5,
                     share=round(rng.uniform(0.4, 0.8), 2))
    if what in ("sym", "spd"):
        n = _log_uniform(rng, 200, 22000)
        return _case(None, entry, what, "f64", rng.choice(["wishart", "matern32", "ntk"]), n,
                     rng.choice([0, 0, 128, 256, 512, 1024]) if n < 9000 else 0, kept=kept,
                     factor=entry == "device" and what == "sym" and rng.random() < 0.3)
    if what == "f32":
        return _case(None, entry, rng.choice(["sym", "spd"]), "f32", "matern32", _log_uniform(rng, 200, 24000), kept=kept)
    if what == "wide":
        return _case(None, entry, rng.choice(["sym", "spd"]), rng.choice(["f32", "bf16", "f16"]), "ntk_narrow",
                     _log_uniform(rng, 200, 16000), wide=True, kept=kept)
    if what == "gen":
        return _case(None, entry, "gen", rng.choice(["f64", "f64", "f32"]), "general", _log_uniform(rng, 200, 9000),
                     kept=kept)
    n = _log_uniform(rng, 200, 8000 if what == "pivot" else 4000)
    return _case(None, entry, what, rng.choice(["f64", "f64", "f32"]), "indefinite", n, kept=kept)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def matrix(case, seed):
    """The matrix on the GPU, in the type it is stored in; from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, kind = case["n"], case["kind"]
    opt = dict(generator=g, dtype=torch.float64, device="cuda")
    if kind == "wishart":                       # G G^T / 2n + 1e-3 I
        f = torch.randn(n, 2 * n, **opt)
        a = f @ f.t() / (2 * n)
        a.diagonal().add_(1e-3)
    elif kind in ("ntk", "ntk_narrow"):         # J J^T / p + shift I with decaying columns, p = n / 4
        p = max(1, n // 4)
        f = torch.randn(n, p, **opt)
        f *= torch.arange(1, p + 1, dtype=torch.float64, device="cuda") ** -0.75
        a = f @ f.t() / p
        # in narrow storage the shift has to stand above the rounding of the entries
        a.diagonal().add_(1e-8 if kind == "ntk" else 0.5 * float(a.diagonal().mean()))
        if case["store"] == "f16":
            a /= float(a.diagonal().mean())     # into the type's range
    elif kind in ("matern32", "se", "general"):
        dim = 8 if kind == "se" else 16
        x = torch.rand(n, dim, **opt)
        a = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        for t in range(dim):                    # squared distances, coordinate by coordinate
            a.addcmul_(x[:, t:t + 1] - x[:, t], x[:, t:t + 1] - x[:, t])
        if kind == "se":
            a.mul_(-1.0 / (2.0 * 0.5 * 0.5)).exp_()
        else:
            a.sqrt_().mul_(math.sqrt(3.0) / 0.3)
            a = (1.0 + a) * torch.exp(-a)
        a.diagonal().add_(1e-6)
        if kind == "matern32":                  # signal variance
            a *= 2.5
        if kind == "general":                   # not symmetric, rows in any order inside each group
            a += torch.randn(n, n, **opt) * (0.25 / math.sqrt(n))
            key = torch.rand(n, **opt) + torch.arange(n, device="cuda") // GROUP
            a = a[torch.argsort(key)]
    elif kind == "indefinite":                  # symmetric noise of norm about 1, diagonal of either sign
        f = torch.randn(n, n, **opt)
        a = (f + f.t()) * (0.35 / math.sqrt(n))
        sign = (torch.rand(n, **opt) < 0.5).to(torch.float64) * 2 - 1
        a.diagonal().add_(sign * (2.0 + 2.0 * torch.rand(n, **opt)))
    else:
        raise ValueError(kind)
    return a.to(STORE[case["store"]]).contiguous()


def _flags(case):
    f = {"sym": 0, "spd": M.FLAG_ASSUME_SPD, "gen": M.FLAG_GENERAL, "pivot": M.FLAG_PIVOT,
         "pivot_block": M.FLAG_PIVOT_BLOCK}[case["form"]]
    return f | (M.FLAG_COMPUTE_F64 if case["wide"] else 0)


def _chooses(case):
    return case["form"] in ("gen", "pivot", "pivot_block")


def _pivots(case, seed):
    """Pivots whose log-determinants follow a scaling law with noise."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    i = torch.arange(1, case["n"] + 1, dtype=torch.float64, device="cuda")
    return 3.0 * i ** -0.6 * torch.exp(0.2 * torch.randn(case["n"], generator=g, dtype=torch.float64, device="cuda"))


def _fit_range(case):
    ns = case["n"] // case["d"]
    return min(100, ns // 10), ns


def prepare(case, seed):
    if case["entry"] == "sequence":
        n0, ns = _fit_range(case)
        at = torch.logspace(math.log10(ns), 6, 1000, dtype=torch.float64, device="cuda")
        return {"case": case, "pivots": _pivots(case, seed), "at": at}
    a = matrix(case, seed)
    n, arith = case["n"], torch.float64 if case["wide"] else STORE[case["store"]]
    s = {"case": case, "flags": _flags(case), "arith": arith}
    if case["entry"] == "host":
        s["packed"] = M.pack_lower_block_columns(a, case["b"])
        s["budget"] = int(case["share"] * n * (n + 1) / 2 * 8)
        s["workspace"] = s["scratch"] = None
        if case["kept"]:
            ws, hs = M.mdet_workspace_query(n, a.dtype, case["b"], s["budget"], overwrite=False, flags=s["flags"])
            s["workspace"] = torch.empty(ws, dtype=torch.uint8, device="cuda")
            s["scratch"] = torch.zeros(max(hs, 1), dtype=torch.uint8)
        return s
    s["a"] = a
    if case["entry"] == "device":
        s["diag"] = torch.empty(n, dtype=arith, device="cuda")
        s["perm"] = torch.empty(n, dtype=torch.int32, device="cuda") if _chooses(case) else None
        s["work"] = torch.empty_like(a) if case["factor"] else None
        s["workspace"] = None
        if case["kept"]:
            ws, _ = M.mdet_workspace_query(n, a.dtype, case["b"], 0, overwrite=case["factor"], flags=s["flags"],
                                           for_device_input=True)
            s["workspace"] = torch.empty(ws, dtype=torch.uint8, device="cuda")
    return s


def run(state):
    case = state["case"]
    if case["entry"] == "sequence":
        n0, ns = _fit_range(case)
        ell = M.mdet_principal_logdets(state["pivots"])
        coef = M.mdet_flodance_fit(ell, case["d"], n0, ns, case["q"])
        return {"ell": ell, "coef": coef, "lhat": M.mdet_flodance_eval(coef, case["q"], state["at"])}
    if case["entry"] == "memdet":
        ld, sign, diag, perm = M.memdet(
            state["a"], assume={"spd": "spd", "gen": "gen"}.get(case["form"], "sym"), block_size=case["b"],
            pivot={"pivot": "leaf", "pivot_block": "block"}.get(case["form"]),
            mixed_precision="float64" if case["wide"] else None)
        out = {"logabsdet": ld, "sign": sign, "diag": diag}
        return dict(out, perm=perm) if _chooses(case) else out
    if case["entry"] == "host":
        diag = torch.empty(case["n"], dtype=state["arith"])
        r = M.mdet_logdet_host(state["packed"], case["n"], case["b"], mem_budget=state["budget"], overwrite=False,
                               flags=state["flags"], diag=diag, workspace=state["workspace"],
                               host_scratch=state["scratch"])
        return {"logabsdet": r.logabsdet, "sign": r.sign, "diag": diag}
    a = state["a"]
    if case["factor"]:
        a = state["work"]
        a.copy_(state["a"])
    r = M.mdet_logdet_device(a, block_size=case["b"], overwrite=case["factor"], flags=state["flags"],
                             diag=state["diag"], workspace=state["workspace"], perm=state["perm"])
    out = {"logabsdet": r.logabsdet, "sign": r.sign, "diag": state["diag"]}
    if state["perm"] is not None:
        out["perm"] = state["perm"]
    if case["factor"]:
        out["factor"] = a
    return out


def work(case):
    n = case["n"]
    if case["entry"] == "sequence":
        rows, cols = _fit_range(case)[1], case["q"] + 3
        return {"bytes": 16 * n + 8 * 2000, "flops": 30 * n + 2 * rows * cols * cols}
    gen = case["form"] == "gen"
    entries = n * n if gen else n * (n + 1) // 2
    arith = 8 if case["wide"] else BYTES[case["store"]]
    out = arith * n + (4 * n if _chooses(case) else 0) + (arith * entries if case["factor"] else 0)
    return {"bytes": entries * BYTES[case["store"]] + out, "flops": (2 if gen else 1) * n ** 3 // 3}


def tolerance(case):
    """About four times what the library is measured to be off `exact` (2-norm, relative)."""
    if case["entry"] == "sequence":             # coefficients: rounding times the fit's condition
        return {"rel": 1e-10}
    if case["store"] == "f32" and not case["wide"]:
        return {"rel": 1e-4}
    # the kernels with a tiny shift: pivots 2e-13, entries of the factor 2e-11 and less
    return {"rel": 5e-11 if case["kind"] in ("se", "ntk") else 1e-12}


# ---------------------------------------------------------------------------
# the same in plain 64-bit torch / numpy
# ---------------------------------------------------------------------------
def _eliminate_symmetric(s):
    """P s P^T = L D L^T, the largest diagonal entry left as the pivot: (L, d, order)."""
    w = s.shape[0]
    order = np.arange(w)
    for j in range(w):
        p = j + int(np.argmax(np.abs(np.diagonal(s)[j:])))
        if p != j:
            s[[j, p]] = s[[p, j]]
            s[:, [j, p]] = s[:, [p, j]]
            order[[j, p]] = order[[p, j]]
        l = s[j + 1:, j] / s[j, j]
        s[j + 1:, j + 1:] -= np.outer(l, s[j, j + 1:])
        s[j + 1:, j] = l
    return np.tril(s, -1) + np.eye(w), np.diagonal(s).copy(), order


def _eliminate_general(s):
    """P s = L U, the largest entry of the column left as the pivot: (L, U, order)."""
    w = s.shape[0]
    order = np.arange(w)
    for j in range(w):
        p = j + int(np.argmax(np.abs(s[j:, j])))
        if p != j:
            s[[j, p]] = s[[p, j]]
            order[[j, p]] = order[[p, j]]
        s[j + 1:, j] /= s[j, j]
        s[j + 1:, j + 1:] -= np.outer(s[j + 1:, j], s[j, j + 1:])
    return np.tril(s, -1) + np.eye(w), np.triu(s), order


def _odd(order):
    seen, odd = np.zeros(len(order), bool), False
    for i in range(len(order)):
        k, length = i, 0
        while not seen[k]:
            seen[k] = True
            k, length = order[k], length + 1
        odd ^= length > 0 and length % 2 == 0
    return odd


def _solve(tri, x, upper, left, unit):
    return torch.linalg.solve_triangular(tri, x, upper=upper, left=left, unitriangular=unit)


def _factor(a, case):
    """(pivots, order, sign of the order, lower factor or None) of the fp64 matrix `a` (overwritten)."""
    n, form = a.shape[0], case["form"]
    # (the library rounds block sizes up to 64 and chooses n / 16 between 256 and 4096)
    block = case["b"] or min(4096, max(256, -(-(n // 16) // 64) * 64))
    step = {"pivot": GROUP, "gen": GROUP, "pivot_block": -(-block // 64) * 64}.get(form, 256)
    diag, order, odd = [], [], False
    for k in range(0, n, step):
        e = min(n, k + step)
        if form in ("sym", "spd"):
            c = torch.linalg.cholesky(a[k:e, k:e].cpu())
            dd = torch.diagonal(c) ** 2
            unit = (c / torch.diagonal(c)).cuda()
            mine = np.arange(e - k)
        elif form == "gen":
            lo, up, mine = _eliminate_general(a[k:e, k:e].cpu().numpy().copy())
            dd = torch.from_numpy(np.diagonal(up).copy())
            odd ^= _odd(mine)
        else:
            lo, dnp, mine = _eliminate_symmetric(a[k:e, k:e].cpu().numpy().copy())
            dd, unit = torch.from_numpy(dnp), torch.from_numpy(lo).cuda()
        diag.append(dd)
        order.append(k + mine)
        idx = torch.from_numpy(mine).cuda()
        if form == "gen":
            if e < n:
                right = _solve(torch.from_numpy(lo).cuda(), a[k:e][idx][:, e:], False, True, True)
                below = _solve(torch.from_numpy(up).cuda(), a[e:, k:e], True, False, False)
                a[e:, e:] -= below @ right
            continue
        dg = dd.cuda()
        if case["factor"]:
            a[k:e, k:e] = torch.tril(unit, -1) + torch.diag(dg)
        if e < n:
            w = _solve(unit.t(), a[e:, k:e][:, idx], True, False, True)          # rows of L D
            l = w / dg
            for r in range(e, n, 8192):
                a[r:r + 8192, e:] -= l[r - e:r - e + 8192] @ w.t()
            if case["factor"]:
                a[e:, k:e] = l
    return torch.cat(diag).numpy(), np.concatenate(order), -1 if odd else 1


def _exact_sequence(case, seed):
    n0, ns = _fit_range(case)
    d, q = case["d"], case["q"]
    ell = np.cumsum(np.log(np.abs(_pivots(case, seed).cpu().numpy())).astype(np.longdouble))
    level = (ell[np.arange(1, ns + 1) * d - 1] / np.arange(1, ns + 1)).astype(np.float64)
    ln0 = level[n0 - 1]
    j = np.arange(n0 + 1, ns + 1, dtype=np.float64)
    lg = torch.lgamma(torch.from_numpy(j + 1.0)).numpy()
    y = j / np.sqrt(j - 1) * (level[n0:] - ln0)
    x = np.stack([np.sqrt(j - 1)] + [-lg * j ** (1.0 - i) / np.sqrt(j - 1) for i in range(1, q + 2)], 1)
    scale = np.linalg.norm(x, axis=0)
    beta = np.linalg.lstsq(x / scale, y, rcond=None)[0]
    res = np.linalg.norm(y - x / scale @ beta)
    beta = beta / scale
    at = np.logspace(math.log10(ns), 6, 1000)
    lgn = torch.lgamma(torch.from_numpy(at + 1.0)).numpy()
    lhat = ln0 + beta[0] * (1 - 1 / at) - sum(beta[i] * at ** -float(i) * lgn for i in range(1, q + 2))
    return {"ell": ell.astype(np.float64), "coef": np.concatenate([beta, [ln0, res]]), "lhat": lhat}


def exact(case, seed):
    if case["entry"] == "sequence":
        return _exact_sequence(case, seed)
    a = matrix(case, seed).to(torch.float64)
    upper = torch.triu(a, 1) if case["factor"] else None       # what the call leaves alone
    diag, order, odd = _factor(a, case)
    out = {"logabsdet": float(np.sum(np.log(np.abs(diag)).astype(np.longdouble))),
           "sign": int(odd * (-1) ** int(np.sum(diag < 0))), "diag": diag}
    if _chooses(case):
        out["perm"] = order
    if case["factor"]:
        out["factor"] = torch.tril(a) + upper
    return out
