"""Dense FP64 contraction and reverse mode where the launch cuts the
contraction into ranges, where monomials of degree above and below 4 share a
step, and at remainders of every tile.

Bound: a sum of m products of at most d + 2 factors, in any order, is within
(m + d + 4) * 2**-53 of the sum of the terms' absolute values.
"""
import numpy as np
import pytest
import torch

import paper_2604_06575_amd as ph

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _basis(rng, n, d, K):
    f = rng.integers(0, n + 1, size=(K, d))
    e = np.zeros((K, n + 1), np.uint8)
    np.add.at(e, (np.arange(K)[:, None], f), 1)
    return np.ascontiguousarray(e[:, :n])


def _values(e, X):
    """Monomial values [K, N] and their derivatives per variable [n, K, N]."""
    K, n = e.shape
    pw = [np.ones_like(X)]
    for _ in range(int(e.max())):
        pw.append(pw[-1] * X)
    pw = np.stack(pw)                                   # [k, N, n]
    v = np.ones((K, X.shape[0]))
    for i in range(n):
        v *= pw[e[:, i], :, i]
    dv = np.zeros((n, K, X.shape[0]))
    for j in range(n):
        ks = np.nonzero(e[:, j])[0]
        p = e[ks, j].astype(np.float64)[:, None] * pw[e[ks, j] - 1, :, j]
        for i in range(n):
            if i != j:
                p = p * pw[e[ks, i], :, i]
        dv[j, ks] = p
    return v, dv


# P, K, N, n, d: one tile with a long contraction (both ranges), remainders of
# one past and one short of the tiles, more than 32 variables, degrees past
# one factor word and past the list, and the smallest shapes
@pytest.mark.parametrize("P,K,N,n,d", [
    (3, 4099, 65, 6, 4), (129, 2063, 127, 5, 6), (64, 130, 2500, 7, 4), (65, 127, 1031, 33, 5),
    (1, 1, 1, 1, 1), (17, 257, 129, 43, 3), (2, 300, 40, 4, 14),
])
def test_dense_fp64_ranges(P, K, N, n, d):
    rng = np.random.default_rng(1000 * P + K + N)
    e = _basis(rng, n, d, K)
    C, X, gY = rng.standard_normal((P, K)), rng.uniform(-1, 1, (N, n)), rng.standard_normal((P, N))
    v, dv = _values(e, X)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    Y = ph.eval_dense(t(e), t(C), t(X)).cpu().numpy()
    dC, dX = (a.cpu().numpy() for a in ph.eval_dense_backward(t(e), t(C), t(X), t(gY)))
    aC, aG, av = np.abs(C), np.abs(gY), np.abs(v)
    assert (np.abs(Y - C @ v) <= 2 * (K + d + 4) * U * (aC @ av)).all()
    assert (np.abs(dC - gY @ v.T) <= 2 * (N + d + 4) * U * (aG @ av.T)).all()
    W, aW = C.T @ gY, aC.T @ aG
    ref = np.einsum("kp,jkp->pj", W, dv)
    bound = np.einsum("kp,jkp->pj", aW, np.abs(dv))
    assert (np.abs(dX - ref) <= 2 * (P + d * K + d + 8) * U * bound).all()


def test_dense_fp64_rows_64():
    """The 64-row tile takes the same ranges."""
    rng = np.random.default_rng(5)
    P, K, N, n, d = 70, 1500, 130, 6, 5
    e = _basis(rng, n, d, K)
    C, X, gY = rng.standard_normal((P, K)), rng.uniform(-1, 1, (N, n)), rng.standard_normal((P, N))
    v, _ = _values(e, X)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    rows = ph.tune_get("dense_f64_rows")
    ph.tune_set("dense_f64_rows", 64)
    try:
        Y = ph.eval_dense(t(e), t(C), t(X)).cpu().numpy()
        dC = ph.eval_dense_backward(t(e), t(C), t(X), t(gY), want_dX=False)[0].cpu().numpy()
    finally:
        ph.tune_set("dense_f64_rows", rows)
    assert (np.abs(Y - C @ v) <= 2 * (K + d + 4) * U * (np.abs(C) @ np.abs(v))).all()
    assert (np.abs(dC - gY @ v.T) <= 2 * (N + d + 4) * U * (np.abs(gY) @ np.abs(v).T)).all()


# dX forms W in a chunk of 8 K min(N, 4096) bytes, dC leaves partial sums of
# 8 P K bytes for each range of points: neither is asked for by a call that
# wants the other alone, and both share memory in a call that wants both
@pytest.mark.parametrize("prec", [ph.POLY_FP64, ph.POLY_SPLIT_BF16])
def test_workspace_of_one_gradient(monkeypatch, prec):
    rng = np.random.default_rng(9)
    P, K, N, n, d = 300, 4000, 3000, 9, 4
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    args = t(_basis(rng, n, d, K)), t(rng.standard_normal((P, K))), t(rng.uniform(-1, 1, (N, n))), t(rng.standard_normal((P, N)))
    asked = []
    make = ph._workspace
    monkeypatch.setattr(ph, "_workspace", lambda nbytes, device: (asked.append(nbytes), make(nbytes, device))[1])
    dC, dX = ph.eval_dense_backward(*args, prec=prec)
    c, _ = ph.eval_dense_backward(*args, prec=prec, want_dX=False)
    _, x = ph.eval_dense_backward(*args, prec=prec, want_dC=False)
    assert torch.equal(c, dC) and torch.equal(x, dX)
    both, only_c, only_x = asked
    assert both == max(only_c, only_x)
    digits = 0 if prec == ph.POLY_FP64 else 5 * 2 * 320 * 3072 + 24 * 4 * K
    assert only_c <= 16 * 8 * P * K * (prec == ph.POLY_FP64) + digits + 32 * K + 2048
    if prec == ph.POLY_FP64:
        assert 8 * K * N <= only_x <= 8 * K * (N + 128) + 64 * 8 * n * (N + 128) + 32 * K + 2048
