"""The work that a user of this library has it do, as cases to be timed.

Every case goes through the public entry points of ``paper_2604_06575_amd``
(products with their simplify, simplify of a polynomial matrix, evaluation,
gradients, reverse mode, the dense shared-set contraction in both precisions,
affine normals).  Sizes are those of the repository's benchmark and tests, or
plain variations of them; :func:`draw` gives further sizes of the same ranges.

``prepare`` makes the inputs on the GPU from the seed alone and ``exact`` gives
the same outputs in plain torch arithmetic in 64 bits, without the library.
Where a result's size depends on which monomials meet, a case has one pattern
of monomials, and the seed renames its variables, shuffles its entries and
terms and draws its coefficients: other inputs with results of the same size.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_06575_amd as ph

DEVICE = "cuda"


def listed():
    return [
        # One small product, the size of an interactive call: the entry point's
        # own latency, launches and the read-back of the output size.
        {"name": "times-small", "op": "times", "pairs": 1, "n": 4, "d": 6, "tmin": 200, "tmax": 200},
        # One product of two large polynomials (25 million raw products), the
        # expand-and-simplify benchmark.
        {"name": "times-large", "op": "times", "pairs": 1, "n": 10, "d": 8, "tmin": 5000, "tmax": 5000},
        # Entrywise product of two 24 x 25 polynomial matrices whose entries
        # have very different sizes.
        {"name": "times-batch", "op": "times", "pairs": 600, "n": 8, "d": 4, "tmin": 6, "tmax": 300},
        # simplify of a 64 x 64 polynomial matrix in 20 variables with repeated
        # monomials in random order (10.7 million terms).
        {"name": "simplify-matrix", "op": "simplify", "entries": 4096, "n": 20, "d": 6, "tmin": 10, "tmax": 20000},
        # The product of two 3 x 3 matrices of degree-4 polynomials.
        {"name": "mtimes", "op": "mtimes", "I": 3, "K": 3, "J": 3, "n": 8, "d": 4, "terms": 300},
        # Values of one product polynomial at a thousand points: a call small
        # enough that its launches are most of it.
        {"name": "eval-small", "op": "eval", "polys": 1, "n": 4, "d": 12, "terms": 1817, "points": 1024},
        # Value and reverse mode (coefficients and points) of a large sparse
        # quartic in 100 variables, as a training step takes them.
        {"name": "quartic-step", "op": "step", "n": 100, "d": 4, "terms": 100000, "points": 8192},
        # Gradients of every entry of a 16 x 16 polynomial matrix in 20
        # variables, the input of matrix-valued optimisation.
        {"name": "grad-matrix", "op": "grad", "entries": 256, "n": 20, "d": 6, "tmin": 10, "tmax": 20000,
         "points": 1000},
        # Value and reverse mode of many polynomials on one shared monomial
        # basis in double precision.
        {"name": "dense-step", "op": "dense", "polys": 500, "n": 20, "d": 4, "points": 5000, "slices": 0},
        # The same through the split BF16 precision, larger.
        {"name": "dense-split-step", "op": "dense", "polys": 1024, "n": 24, "d": 4, "points": 8192, "slices": 5},
        # Affine-normal directions of a sparse quartic at many points, as a
        # descent method over a population of iterates takes them ...
        {"name": "affine", "op": "affine", "n": 64, "support": 3, "per_var": 4, "points": 4096},
        # ... and of one in more variables at fewer points.
        {"name": "affine-wide", "op": "affine", "n": 160, "support": 3, "per_var": 4, "points": 256},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: an operation and sizes of the ranges the listed ones stand for."""
    op = rng.choice(["times", "times", "simplify", "mtimes", "eval", "step", "grad", "dense", "affine"])
    if op == "times":
        if rng.random() < 0.5:
            n, d = rng.randint(4, 12), rng.randint(4, 8)
            t = min(_log_int(rng, 30, 5000), math.comb(n + d, d))
            return {"op": op, "pairs": 1, "n": n, "d": d, "tmin": t, "tmax": t}
        n, d = rng.randint(3, 10), rng.randint(3, 5)
        hi = min(_log_int(rng, 30, 400), math.comb(n + d, d))
        return {"op": op, "pairs": _log_int(rng, 2, 600), "n": n, "d": d, "tmin": _log_int(rng, 1, hi), "tmax": hi}
    if op == "simplify":
        return {"op": op, "entries": _log_int(rng, 1, 4096), "n": rng.randint(5, 24), "d": rng.randint(4, 7),
                "tmin": 10, "tmax": _log_int(rng, 100, 20000)}
    if op == "mtimes":
        n, d = rng.randint(3, 10), rng.randint(2, 5)
        return {"op": op, "I": rng.randint(1, 5), "K": rng.randint(1, 5), "J": rng.randint(1, 5), "n": n, "d": d,
                "terms": min(_log_int(rng, 5, 400), math.comb(n + d, d))}
    if op == "eval":
        n, d = rng.randint(3, 30), rng.randint(2, 12)
        return {"op": op, "polys": _log_int(rng, 1, 64), "n": n, "d": d,
                "terms": min(_log_int(rng, 20, 5000), math.comb(n + d, d)), "points": _log_int(rng, 17, 8192)}
    if op == "step":
        n, d = _log_int(rng, 8, 120), rng.randint(3, 5)
        return {"op": op, "n": n, "d": d, "terms": min(_log_int(rng, 200, 100000), math.comb(n + d, d) // 2),
                "points": _log_int(rng, 100, 8192)}
    if op == "grad":
        return {"op": op, "entries": _log_int(rng, 1, 256), "n": rng.randint(5, 24), "d": rng.randint(3, 7),
                "tmin": 10, "tmax": _log_int(rng, 50, 20000), "points": _log_int(rng, 64, 1000)}
    if op == "dense":
        return {"op": op, "polys": _log_int(rng, 64, 1024), "n": rng.randint(8, 24), "d": rng.randint(3, 4),
                "points": _log_int(rng, 256, 8192), "slices": rng.choice([0, 0, 4, 5])}
    n = _log_int(rng, 12, 200)
    return {"op": op, "n": n, "support": rng.randint(2, 3), "per_var": rng.randint(3, 5),
            "points": max(16, min(4096, int(_log_int(rng, 64, 4096) * min(1.0, (64 / n) ** 3))))}


# -------------------------------------------------------------------- inputs

class _Rng:
    """torch draws on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEVICE)
        self.g.manual_seed(int(seed))

    def rand(self, *shape):
        return torch.rand(*shape, generator=self.g, device=DEVICE, dtype=torch.float64)

    def randn(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEVICE, dtype=torch.float64)

    def randint(self, lo, hi, shape):
        return torch.randint(lo, hi, shape, generator=self.g, device=DEVICE)

    def points(self, count, n, r=1.0):
        return (self.rand(count, n) * 2.0 - 1.0) * r


def _factor_lists(r, n, d, m):
    """m monomials drawn uniformly over those of degree <= d in n variables, as
    sorted lists of d factors (the value n stands for the factor 1): d distinct
    slots among n + d, less their rank."""
    got = []
    have = 0
    while have < m:
        want = min((m - have) * 2 + 64, 8_000_000)
        s = r.randint(0, n + d, (want, d)).sort(dim=1).values
        if d > 1:
            s = s[(s[:, 1:] > s[:, :-1]).all(dim=1)]
        got.append(s - torch.arange(d, device=DEVICE))
        have += got[-1].shape[0]
    return torch.cat(got)[:m]


def _exps(lists, n):
    """uint8 exponent rows of factor lists."""
    e = torch.zeros((lists.shape[0], n + 1), dtype=torch.uint8, device=DEVICE)
    e.scatter_add_(1, lists, torch.ones_like(lists, dtype=torch.uint8))
    return e[:, :n].contiguous()


def _all_lists(n, d):
    """Every monomial of degree <= d in n variables, as sorted factor lists."""
    return torch.combinations(torch.arange(n + 1, device=DEVICE), d, with_replacement=True)


def _distinct(r, n, d, m):
    """m distinct monomials of degree <= d, in random order."""
    total = math.comb(n + d, d)
    if total <= 200_000:
        every = _all_lists(n, d)
        return _exps(every[torch.randperm(total, generator=r.g, device=DEVICE)[:m]], n)
    weights = torch.tensor([(n + 1) ** k for k in range(d)], dtype=torch.int64, device=DEVICE)
    lists = _factor_lists(r, n, d, m)
    while True:
        key = (lists * weights).sum(dim=1)
        order = key.argsort(stable=True)
        first = torch.ones(len(key), dtype=torch.bool, device=DEVICE)
        first[1:] = key[order][1:] != key[order][:-1]
        lists = lists[order[first].sort().values]
        if lists.shape[0] >= m:
            return _exps(lists[:m], n)
        lists = torch.cat([lists, _factor_lists(r, n, d, m // 4 + 64)])


def _sizes(r, count, tmin, tmax):
    """Log-uniform entry sizes on [tmin, tmax] and their row pointer (host)."""
    u = r.rand(count).cpu().numpy()
    t = np.clip(np.floor(np.exp(math.log(tmin) + u * math.log(max(tmax, 1) / tmin))), tmin, tmax).astype(np.int64)
    rp = np.zeros(count + 1, np.int64)
    np.cumsum(t, out=rp[1:])
    return rp


def _batch(n, max_exp, rp, exps, coefs):
    return ph.Batch(n, max_exp, torch.from_numpy(rp).to(DEVICE), rp, exps, coefs)


def _shuffled(r, n, d, rp, exps, names, entries):
    """The pattern (rp, exps) with its variables renamed, its entries in the
    order `entries`, each entry's terms in random order, and N(0,1) coefficients."""
    sizes = torch.from_numpy(np.diff(rp)).to(DEVICE)
    rank = torch.empty_like(entries)
    rank[entries] = torch.arange(len(entries), device=DEVICE)
    place = torch.repeat_interleave(rank, sizes).to(torch.float64) + r.rand(exps.shape[0])
    exps = exps[place.argsort()][:, names].contiguous()
    rp = np.zeros(len(entries) + 1, np.int64)
    np.cumsum(sizes[entries].cpu().numpy(), out=rp[1:])
    return _batch(n, d, rp, exps, r.randn(exps.shape[0]))


def _distinct_pattern(r, case, count):
    """Row pointer and rows of `count` entries, distinct monomials in each."""
    rp = _sizes(r, count, case["tmin"], case["tmax"])
    n, d = case["n"], case["d"]
    if count == 1:
        return rp, _distinct(r, n, d, int(rp[-1]))
    every = _exps(_all_lists(n, d), n)
    return rp, torch.cat([every[torch.randperm(every.shape[0], generator=r.g, device=DEVICE)[:int(t)]]
                          for t in np.diff(rp)])


def _repeating_pattern(r, case):
    rp = _sizes(r, case["entries"], case["tmin"], case["tmax"])
    T = int(rp[-1])
    return rp, torch.cat([_exps(_factor_lists(r, case["n"], case["d"], min(2_000_000, T - o)), case["n"])
                          for o in range(0, T, 2_000_000)])


def _sparse_quartic(r, n, support, m):
    """The affine-normal family: m distinct quartic monomials of support 3
    (exponents 2, 1, 1) or 2 (a, 4 - a), plus sum x_i^2."""
    e = torch.zeros((0, n), dtype=torch.uint8, device=DEVICE)
    while e.shape[0] < m:
        k = m * 2 + 64
        v = r.rand(k, n).argsort(dim=1)[:, :support]
        if support == 3:
            x = torch.tensor([2, 1, 1], dtype=torch.uint8, device=DEVICE).expand(k, 3)
        else:
            a = r.randint(1, 4, (k, 1))
            x = torch.cat([a, 4 - a], dim=1).to(torch.uint8)
        e = torch.cat([e, torch.zeros((k, n), dtype=torch.uint8, device=DEVICE).scatter_(1, v, x)])
        e = torch.unique(e, dim=0)
        e = e[torch.randperm(e.shape[0], generator=r.g, device=DEVICE)]
    e = torch.cat([e[:m], 2 * torch.eye(n, dtype=torch.uint8, device=DEVICE)])
    return e.contiguous(), torch.cat([r.randn(m), torch.ones(n, dtype=torch.float64, device=DEVICE)])


def _one(n, d, exps, coefs):
    return _batch(n, d, np.array([0, exps.shape[0]], np.int64), exps, coefs)


def prepare(case, seed):
    r, op, n = _Rng(seed), case["op"], case["n"]
    pattern, names = _Rng(20260321), torch.randperm(n, generator=r.g, device=DEVICE)
    s = {"op": op}
    if op == "times":
        order = torch.randperm(case["pairs"], generator=r.g, device=DEVICE)
        for k in ("a", "b"):
            s[k] = _shuffled(r, n, case["d"], *_distinct_pattern(pattern, case, case["pairs"]), names, order)
    elif op in ("simplify", "grad"):
        order = torch.randperm(case["entries"], generator=r.g, device=DEVICE)
        s["a"] = _shuffled(r, n, case["d"], *_repeating_pattern(pattern, case), names, order)
        if op == "grad":
            s["X"] = r.points(case["points"], n)
    elif op == "mtimes":
        s["shape"] = (case["I"], case["K"], case["J"])
        c = dict(case, tmin=case["terms"], tmax=case["terms"])
        for k, count in (("a", case["I"] * case["K"]), ("b", case["K"] * case["J"])):
            s[k] = _shuffled(r, n, case["d"], *_distinct_pattern(pattern, c, count), names,
                             torch.arange(count, device=DEVICE))
    elif op == "eval":
        rp = np.arange(case["polys"] + 1, dtype=np.int64) * case["terms"]
        e = torch.cat([_distinct(r, n, case["d"], case["terms"]) for _ in range(case["polys"])])
        s["a"] = _batch(n, case["d"], rp, e, r.randn(int(rp[-1])))
        s["X"] = r.points(case["points"], n)
    elif op == "step":
        e = _distinct(r, n, case["d"], case["terms"])
        s["coefs"] = r.randn(case["terms"]).requires_grad_()
        s["a"] = _one(n, case["d"], e, s["coefs"].detach())
        s["X"] = r.points(case["points"], n).requires_grad_()
        s["gY"] = r.randn(1, case["points"])
    elif op == "dense":
        s["basis"] = _exps(_all_lists(n, case["d"]), n)
        s["C"] = r.randn(case["polys"], s["basis"].shape[0]).requires_grad_()
        s["X"] = r.points(case["points"], n).requires_grad_()
        s["gY"] = r.randn(case["polys"], case["points"])
        s["prec"] = (ph.POLY_SPLIT_BF16, case["slices"]) if case["slices"] else (ph.POLY_FP64, 5)
    else:
        e, c = _sparse_quartic(r, n, case["support"], case["per_var"] * n)
        s["a"] = _one(n, 4, e, c)
        # the locally convex regime, where every tangent block is positive definite
        s["X"] = r.points(case["points"], n, 0.1)
    return s


# ---------------------------------------------------------------------- pass

def _terms(b):
    return {"row_ptr": b.row_ptr, "exps": b.exps, "coefs": b.coefs}


def run(s):
    op = s["op"]
    if op == "times":
        return _terms(ph.mul(s["a"], s["b"]))
    if op == "simplify":
        return _terms(ph.simplify(s["a"]))
    if op == "mtimes":
        return _terms(ph.mtimes(s["a"], s["b"], *s["shape"]))
    if op == "eval":
        return ph.eval(s["a"], s["X"])
    if op == "grad":
        return ph.grad(s["a"], s["X"])
    if op == "step":
        Y = ph.PolyEval.apply(s["coefs"], s["X"], s["a"])
        dC, dX = torch.autograd.grad(Y, (s["coefs"], s["X"]), s["gY"])
        return {"Y": Y.detach(), "dC": dC, "dX": dX}
    if op == "dense":
        Y = ph.PolyEvalDense.apply(s["C"], s["X"], s["basis"], *s["prec"])
        dC, dX = torch.autograd.grad(Y, (s["C"], s["X"]), s["gY"])
        return {"Y": Y.detach(), "dC": dC, "dX": dX}
    D, g = ph.affine_normal(s["a"], s["X"], reg=1e-8)
    return {"D": D, "gnorm": g}


# ---------------------------------------------------------------------- work

def _mean_size(tmin, tmax):
    return float(tmin) if tmin == tmax else (tmax - tmin) / math.log(tmax / tmin)


def _occupied(balls, cells):
    """Expected number of distinct monomials among `balls` draws."""
    return cells * -math.expm1(-balls / cells)


def work(case):
    """Bytes and flops that the case cannot do without: inputs read once,
    outputs written once; one multiplication and one addition per raw product,
    d multiplications and one addition per term and point."""
    op, n, d = case["op"], case["n"], case.get("d", 4)
    row = n + 8
    if op == "times":
        m = _mean_size(case["tmin"], case["tmax"])
        raw = m * m
        out = min(raw, _occupied(raw, math.comb(n + 2 * d, 2 * d)))
        return {"bytes": case["pairs"] * (2 * m + out) * row, "flops": case["pairs"] * 2 * raw}
    if op == "simplify":
        m = _mean_size(case["tmin"], case["tmax"])
        return {"bytes": case["entries"] * (m + _occupied(m, math.comb(n + d, d))) * row,
                "flops": case["entries"] * m}
    if op == "mtimes":
        I, K, J, t = case["I"], case["K"], case["J"], case["terms"]
        raw = K * t * t
        out = min(raw, _occupied(raw, math.comb(n + 2 * d, 2 * d)))
        return {"bytes": ((I * K + K * J) * t + I * J * out) * row, "flops": 2.0 * I * J * raw}
    if op == "eval":
        T, N = case["polys"] * case["terms"], case["points"]
        return {"bytes": T * row + 8 * N * (n + case["polys"]), "flops": float(T) * N * (d + 1)}
    if op == "step":
        T, N = case["terms"], case["points"]
        return {"bytes": T * (row + 8) + 8 * N * (2 * n + 2), "flops": float(T) * N * (d + 1 + d * (d + 1) + d + 1)}
    if op == "grad":
        T, N = case["entries"] * _mean_size(case["tmin"], case["tmax"]), case["points"]
        return {"bytes": T * row + 8 * N * n * (1 + case["entries"]), "flops": float(T) * N * d * (d + 1)}
    if op == "dense":
        P, K, N = case["polys"], math.comb(n + d, d), case["points"]
        S = case["slices"]
        return {"bytes": K * n + 8 * (2 * P * K + 2 * P * N + 2 * N * n),
                "flops": 6.0 * P * K * N * (S * (S + 1) // 2 if S else 1)}
    N, T = case["points"], n * (case["per_var"] + 1)
    return {"bytes": T * row + 8 * N * (2 * n + 1), "flops": float(N) * (2 * (n - 1) ** 3 + 18 * n * n + 100 * T)}


# --------------------------------------------------------------------- exact

def _keys(e, radix):
    w = torch.tensor([radix ** (e.shape[1] - 1 - i) for i in range(e.shape[1])], dtype=torch.int64, device=DEVICE)
    return (e.to(torch.int64) * w).sum(dim=1)


def _rows(keys, n, radix):
    return torch.stack([(keys // radix ** (n - 1 - i)) % radix for i in range(n)], dim=1).to(torch.uint8)


def _merged(n, parts):
    """row_ptr, exps and coefs of a batch from per-entry (keys, values), merged;
    or, where a key passes 64 bits, from per-entry (rows, values)."""
    rp, es, cs = [0], [], []
    for radix, k, v in parts:
        if radix is None:
            u, inv = torch.unique(k, dim=0, return_inverse=True)
        else:
            u, inv = torch.unique(k, return_inverse=True)
        c = torch.zeros(u.shape[0], dtype=torch.float64, device=DEVICE).index_add_(0, inv, v)
        keep = c != 0
        u, c = u[keep], c[keep]
        es.append(u.to(torch.uint8) if radix is None else _rows(u, n, radix))
        cs.append(c)
        rp.append(rp[-1] + int(c.shape[0]))
    return {"row_ptr": torch.tensor(rp, dtype=torch.int64), "exps": torch.cat(es), "coefs": torch.cat(cs)}


def _entry(b, p):
    lo, hi = int(b.row_ptr_host[p]), int(b.row_ptr_host[p + 1])
    return b.exps[lo:hi], b.coefs[lo:hi]


def _product(a, p, b, q, radix):
    (ea, ca), (eb, cb) = _entry(a, p), _entry(b, q)
    k = (_keys(ea, radix)[:, None] + _keys(eb, radix)[None, :]).reshape(-1)
    return k, (ca[:, None] * cb[None, :]).reshape(-1)


def _monomials(e, X):
    """V[t, pt] of exponent rows at points."""
    v = torch.ones((e.shape[0], X.shape[0]), dtype=torch.float64, device=DEVICE)
    top = int(e.max()) if e.numel() else 0
    pw = torch.stack([X.T ** k for k in range(top + 1)])          # [k, n, N]
    for i in range(e.shape[1]):
        v *= pw[e[:, i].long(), i]
    return v


def _chunks(T, N):
    step = max(1, int(5e7 // max(N, 1)))
    return [(o, min(o + step, T)) for o in range(0, T, step)]


def _tangent_basis(g):
    """Orthonormal basis of the complement of each row of g: the last columns
    of a complete QR factorisation that starts with it."""
    Q, _ = torch.linalg.qr(g[:, :, None], mode="complete")
    return Q[:, :, 1:]


def _affine(e, c, X, reg):
    """nu = Q_T tau - e with A = Q_T' H Q_T + reg I, a_i = tr(A^-1 d_i H_T) and
    tau = A^-1 (h - |g| / (n + 1) a), point by point."""
    N, n = X.shape
    T = e.shape[0]
    lists = torch.full((T, 4), n, dtype=torch.int64, device=DEVICE)
    host = e.cpu().numpy()
    for t in range(T):
        f = np.repeat(np.arange(n), host[t])
        lists[t, :len(f)] = torch.from_numpy(f).to(DEVICE)
    x1 = torch.cat([X, torch.ones((N, 1), dtype=torch.float64, device=DEVICE)], dim=1)
    D, gn = [], []
    for o in range(0, N, 256):
        x = x1[o:o + 256]
        m = x.shape[0]
        f = x[:, lists]                                            # [m, T, 4]
        g = torch.zeros((m, n + 1), dtype=torch.float64, device=DEVICE)
        H = torch.zeros((m, (n + 1) * (n + 1)), dtype=torch.float64, device=DEVICE)
        for i in range(4):
            r1 = [k for k in range(4) if k != i]
            g.index_add_(1, lists[:, i], c * f[:, :, r1].prod(dim=2))
            for j in r1:
                r2 = [k for k in r1 if k != j]
                H.index_add_(1, lists[:, i] * (n + 1) + lists[:, j], c * f[:, :, r2].prod(dim=2))
        g, H = g[:, :n], H.reshape(m, n + 1, n + 1)[:, :n, :n]
        norm = g.norm(dim=1)
        unit = g / norm[:, None]
        Q = _tangent_basis(unit)
        A = Q.mT @ H @ Q + reg * torch.eye(n - 1, dtype=torch.float64, device=DEVICE)
        M = torch.zeros((m, n + 1, n + 1), dtype=torch.float64, device=DEVICE)
        M[:, :n, :n] = Q @ torch.linalg.solve(A, Q.mT)
        M = M.reshape(m, -1)
        w = torch.zeros((m, n + 1), dtype=torch.float64, device=DEVICE)
        for i in range(4):
            for j in range(4):
                for k in range(4):
                    if i != j and j != k and i != k:
                        rest = 6 - i - j - k
                        pair = M[:, lists[:, i] * (n + 1) + lists[:, j]]
                        w.index_add_(1, lists[:, k], c * pair * f[:, :, rest])
        a = (Q.mT @ w[:, :n, None])[:, :, 0]
        h = (Q.mT @ (H @ unit[:, :, None]))[:, :, 0]
        tau = torch.linalg.solve(A, h - norm[:, None] / (n + 1) * a)
        D.append((Q @ tau[:, :, None])[:, :, 0] - unit)
        gn.append(norm)
    return torch.cat(D), torch.cat(gn)


def exact(case, seed):
    s, op, n = prepare(case, seed), case["op"], case["n"]
    a = s.get("a")
    if op == "times":
        radix = 2 * case["d"] + 1
        return _merged(n, [(radix, *_product(a, p, s["b"], p, radix)) for p in range(a.npolys)])
    if op == "mtimes":
        radix, (I, K, J) = 2 * case["d"] + 1, s["shape"]
        parts = []
        for i in range(I):
            for j in range(J):
                raw = [_product(a, i * K + k, s["b"], k * J + j, radix) for k in range(K)]
                parts.append((radix, torch.cat([k for k, _ in raw]), torch.cat([v for _, v in raw])))
        return _merged(n, parts)
    if op == "simplify":
        radix = case["d"] + 1
        fits = radix ** n < 2 ** 62
        return _merged(n, [(radix if fits else None, _keys(e, radix) if fits else e, c)
                           for e, c in (_entry(a, p) for p in range(a.npolys))])
    if op == "eval":
        return torch.stack([(_monomials(e, s["X"]) * c[:, None]).sum(dim=0)
                            for e, c in (_entry(a, p) for p in range(a.npolys))])
    if op == "grad":
        X = s["X"]
        G = torch.zeros((a.npolys, X.shape[0], n), dtype=torch.float64, device=DEVICE)
        for p in range(a.npolys):
            e, c = _entry(a, p)
            for lo, hi in _chunks(e.shape[0], X.shape[0]):
                G[p] += _monomials(e[lo:hi], X).T @ (c[lo:hi, None] * e[lo:hi]) / X
        return G
    if op == "step":
        X, c, gY = s["X"].detach(), s["coefs"].detach(), s["gY"]
        Y, dX, dC = torch.zeros_like(gY), torch.zeros_like(X), []
        for lo, hi in _chunks(c.shape[0], X.shape[0]):
            v = _monomials(a.exps[lo:hi], X)
            Y[0] += c[lo:hi] @ v
            dC.append(v @ gY[0])
            dX += (v.T @ (c[lo:hi, None] * a.exps[lo:hi])) * gY[0][:, None] / X
        return {"Y": Y, "dC": torch.cat(dC), "dX": dX}
    if op == "dense":
        X, C, gY = s["X"].detach(), s["C"].detach(), s["gY"]
        Y, dX, dC = torch.zeros_like(gY), torch.zeros_like(X), []
        basis = s["basis"]
        for lo, hi in _chunks(basis.shape[0], X.shape[0]):
            v = _monomials(basis[lo:hi], X)
            Y += C[:, lo:hi] @ v
            dC.append(gY @ v.T)
            dX += ((C[:, lo:hi].T @ gY) * v).T @ basis[lo:hi].to(torch.float64) / X
        return {"Y": Y, "dC": torch.cat(dC, dim=1), "dX": dX}
    D, gn = _affine(a.exps, a.coefs, s["X"], 1e-8)
    return {"D": D, "gnorm": gn}
