"""Sparse evaluation and reverse mode of long batches of low degree (the
coordinates in registers): at the variable counts where the registers and the
tile's rows change, in every degree class, and at ranges around the 8, 16 and
32 terms of a step beside long ones.

Bound: a sum of m products of at most d + 3 factors, in any order, is within
(m + d + 5) * 2**-53 of the sum of the terms' absolute values.
"""
import numpy as np
import pytest
import torch

import paper_2604_06575_amd as ph

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _batch(rng, n, d, sizes):
    """Factor lists padded with n, and the exponent rows.  Variables 1 to 6
    occur in few terms and variable 2 in none; the last one often, also twice."""
    T = sum(sizes)
    f = rng.integers(0, n, size=(T, d))
    f[:, :2] = np.where(rng.random((T, 2)) < 0.2, n - 1, f[:, :2])
    if n > 7:
        f[(f > 0) & (f < 7)] = n - 2
        for v, m in ((1, 1), (3, 7), (4, 8), (5, 33), (6, 65)):
            f[rng.choice(T, m, replace=False), 0] = v
    f[np.arange(d)[None, :] >= rng.integers(0, d + 1, size=T)[:, None]] = n
    f[-1, :] = rng.integers(0, n, size=d)                               # one term of the full degree
    f.sort(axis=1)
    e = np.zeros((T, n + 1), np.uint8)
    np.add.at(e, (np.arange(T)[:, None], f), 1)
    rp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return f, np.ascontiguousarray(e[:, :n]), rp, rng.standard_normal(T)


def _padded(X):
    return np.concatenate([X, np.ones((X.shape[0], 1))], axis=1).astype(np.longdouble)


CASES = [(4, 8), (23, 2), (24, 3), (55, 4), (56, 5), (100, 6), (112, 4), (112, 7), (55, 8), (113, 4), (40, 9), (129, 3),
         (200, 4)]


@pytest.mark.parametrize("n,d", CASES)
def test_eval(n, d):
    rng = np.random.default_rng(100 * n + d)
    sizes = [0, 1, 15, 16, 18, 33, 0, 64, 131, 8191]
    f, e, rp, c = _batch(rng, n, d, sizes)
    N = 65601
    X = rng.uniform(-1, 1, (N, n))
    X[3, 0], X[70, n - 1], X[N - 1, 0] = np.inf, np.nan, -np.inf
    b = ph.batch_from_numpy(rp, e, c)
    t = torch.from_numpy(X).cuda()
    Y = ph.eval(b, t).cpu().numpy().reshape(-1, N)
    assert np.array_equal(Y, ph.eval(b, t).cpu().numpy().reshape(-1, N), equal_nan=True)
    pts = np.concatenate([np.arange(0, 3), np.arange(60, 70), np.arange(71, N - 1, 999), np.arange(N - 70, N - 1)])
    v = c * np.prod(_padded(X[pts])[:, f], axis=2)                       # [points, T]
    for p, m in enumerate(sizes):
        s = v[:, rp[p]:rp[p + 1]]
        assert np.all(np.abs(Y[p, pts] - s.sum(1)) <= (m + d + 5) * U * np.abs(s).sum(1)), p
    # one term past the degrees of the fast forms: the other polynomials are
    # evaluated by the general kernel, to the same bits
    e2 = e.copy()
    e2[-1, 0] += 9
    Y2 = ph.eval(ph.batch_from_numpy(rp, e2, c), t).cpu().numpy().reshape(-1, N)
    assert np.array_equal(Y[:-1], Y2[:-1], equal_nan=True)


@pytest.mark.parametrize("n,d", [c for c in CASES if c[0] > 7])
def test_dx(n, d):
    rng = np.random.default_rng(200 * n + d)
    sizes = [20000, 9001]
    f, e, rp, c = _batch(rng, n, d, sizes)
    N, P = 1281, len(sizes)
    X, gY = rng.uniform(-1, 1, (N, n)), rng.standard_normal((P, N))
    gX, _ = ph.eval_backward(ph.batch_from_numpy(rp, e, c), torch.from_numpy(X).cuda(), torch.from_numpy(gY).cuda(),
                             want_dX=True, want_dC=False)
    pts = np.array([0, 1, 63, 64, 127, 128, 640, 1279, 1280])
    x = _padded(X[pts])[:, f]                                           # [points, T, d]
    g = np.repeat(gY[:, pts], sizes, axis=0).T * c                      # [points, T]
    ref, mag = np.zeros((n + 1, len(pts)), np.longdouble), np.zeros((n + 1, len(pts)), np.longdouble)
    cnt = np.zeros((n + 1, 1))
    for k in range(d):                                                  # the derivative in the k-th factor
        q = (g * np.prod(np.delete(x, k, axis=2), axis=2)).T            # [T, points]
        np.add.at(ref, f[:, k], q)
        np.add.at(mag, f[:, k], np.abs(q))
        np.add.at(cnt, f[:, k], 1)
    got = gX.cpu().numpy().T[:, pts]
    assert np.all(np.abs(got - ref[:n]) <= (cnt[:n] + d + 5) * U * mag[:n])


@pytest.mark.parametrize("n,d", CASES)
def test_dc(n, d):
    rng = np.random.default_rng(300 * n + d)
    sizes = [0, 3, 20001, 64, 135, 9007]
    f, e, rp, c = _batch(rng, n, d, sizes)
    N, P = 2561, len(sizes)
    X, gY = rng.uniform(-1, 1, (N, n)), rng.standard_normal((P, N))
    b, x, g = ph.batch_from_numpy(rp, e, c), torch.from_numpy(X).cuda(), torch.from_numpy(gY).cuda()
    _, dC = ph.eval_backward(b, x, g, want_dX=False, want_dC=True)
    gX, dC2 = ph.eval_backward(b, x, g)
    assert torch.equal(dC, dC2)
    t = np.unique(np.concatenate([np.arange(300), rp[:-1], rp[1:-1] - 1, np.arange(rp[3] - 70, rp[3] + 70),
                                  np.arange(rp[-1] - 130, rp[-1]), rng.integers(0, rp[-1], 300)]))
    v = np.prod(_padded(X)[:, f[t]], axis=2)                             # [N, terms]
    v = v * gY[np.searchsorted(rp, t, side="right") - 1].T
    got = dC.cpu().numpy()[t]
    assert np.all(np.abs(got - v.sum(0)) <= (N + d + 5) * U * np.abs(v).sum(0))


# more tiles of points than the partial sums of one pass (256 MB) have room
# for: 2,344 tiles of 128 points, 1,677 a pass; a degree past the register form
@pytest.mark.parametrize("d", [3, 6, 9])
def test_dc_in_passes(d):
    rng = np.random.default_rng(400 + d)
    n, N = 10, 300_001
    f, e, rp, c = _batch(rng, n, d, [20001, 7])
    X, gY = rng.uniform(-1, 1, (N, n)), rng.standard_normal((2, N))
    _, dC = ph.eval_backward(ph.batch_from_numpy(rp, e, c), torch.from_numpy(X).cuda(), torch.from_numpy(gY).cuda(),
                             want_dX=False, want_dC=True)
    t = np.concatenate([rng.integers(0, rp[-1], 12), [0, 20000, 20001, 20007]])
    x = _padded(X)
    for k in t:
        v = np.prod(x[:, f[k]], axis=1) * gY[int(k >= rp[1])]
        assert np.abs(dC[k].item() - v.sum()) <= (N + d + 5) * U * np.abs(v).sum(), k


def test_host_offsets_beyond_the_device_s():
    """The library plans from the host's offsets and sums by the device's: a
    batch whose host copy is only a bound is evaluated whole."""
    rng = np.random.default_rng(500)
    n, d, N = 20, 3, 1025
    f, e, rp, c = _batch(rng, n, d, [100_000])
    X = torch.from_numpy(rng.uniform(-1, 1, (N, n))).cuda()
    for T in (0, 1, 100, 5000, 99_999):
        b = ph.batch_from_numpy(rp, e, c)
        b.row_ptr.copy_(torch.tensor([0, T]))
        for k in range(4):   # values not written would be these
            Y = torch.full((1, N), np.nan, dtype=torch.float64, device="cuda")
        del Y
        got = ph.eval(b, X).reshape(-1)
        v = c[:T] * np.prod(_padded(X.cpu().numpy()[:50])[:, f[:T]], axis=2)
        assert np.all(np.abs(got.cpu().numpy()[:50] - v.sum(1)) <= (T + d + 5) * U * np.abs(v).sum(1)), T
