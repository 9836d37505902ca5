"""Derivative formation at the counts where a term's variables, the lanes of a
wave and the chunks of a polynomial run over: terms of none, eight, nine and all
variables, rows that are no whole words or not staged, and one term more or
less than a wave and a workgroup.  Bit for bit: rows, order and coefficients."""
import numpy as np
import pytest
import torch

import paper_2604_06575_amd as ph

pytestmark = pytest.mark.gpu


def _jacobian(rp, e, c):
    n = e.shape[1]
    E, C, sizes = [], [], [0]
    for p in range(len(rp) - 1):
        ep, cp = e[rp[p]:rp[p + 1]], c[rp[p]:rp[p + 1]]
        for j in range(n):
            k = np.nonzero(ep[:, j])[0]
            d = ep[k].copy()
            d[:, j] -= 1
            E.append(d)
            C.append(cp[k] * ep[k, j].astype(np.float64))
            sizes.append(len(k))
    return np.cumsum(sizes), np.concatenate(E), np.concatenate(C)


@pytest.mark.parametrize("n,most", [(1, 1), (3, 3), (8, 8), (9, 8), (12, 8), (16, 9), (17, 9), (66, 9), (100, 4), (128, 8), (130, 5), (255, 8)])
def test_formation(n, most):
    rng = np.random.default_rng(10 * n + most)
    sizes = [0, 1, 63, 65, 255, 256, 257, 0, 1030]
    T = sum(sizes)
    e = np.zeros((T, n), np.uint8)
    for t in range(T):
        v = rng.choice(n, min(n, int(rng.integers(0, most + 1))), replace=False)
        e[t, v] = rng.integers(1, 4, len(v))
    rp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    c = rng.standard_normal(T)
    J = ph.jacobian(ph.batch_from_numpy(rp, e, c))
    jrp, je, jc = ph.batch_to_numpy(J)
    rrp, re, rc = _jacobian(rp, e, c)
    assert np.array_equal(jrp, rrp) and np.array_equal(je, re)
    assert np.array_equal(jc.view(np.uint64), rc.view(np.uint64))
    X = rng.uniform(-1, 1, (5, n))
    if n <= 12:                                  # Hessian entries are formed from these
        H = ph.hess(ph.batch_from_numpy(rp, e, c), torch.from_numpy(X).cuda()).cpu().numpy()
        hrp, he, hc = _jacobian(rrp, re, rc)
        for i in range(len(hrp) - 1):
            v = hc[hrp[i]:hrp[i + 1], None] * np.prod(X.T[None] ** he[hrp[i]:hrp[i + 1], :, None], axis=1)
            p, jk = divmod(i, n * n)
            bound = (len(v) + 3 * n + 8) * 2.0 ** -52 * np.abs(v).sum(0)
            assert np.all(np.abs(H[p, :, jk // n, jk % n] - v.sum(0)) <= bound)
