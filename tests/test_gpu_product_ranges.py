"""Products formed on a dense range of monomials (the route that mul and
mtimes take once both operands' degrees are known): bit for bit the oracle's,
and the general route's, at the edges of chunks, ranges and steps."""
import itertools
import math

import numpy as np
import pytest
import torch

import oracle
import workloads as W
import paper_2604_06575_amd as ph

pytestmark = pytest.mark.gpu


def _poly(rng, n, d, t, repeats=False):
    e = W.monomials_with_replacement(rng, n, d, t) if repeats else W.distinct_monomials(rng, n, d, t)
    c = rng.standard_normal(t)
    return e, c


def _batch(polys, n, me):
    rp, e, c = W.csr_from_list(polys, n)
    return ph.batch_from_numpy(rp, e, c, n=n, max_exp=me)


def _same(got, want):
    rp, e, c = ph.batch_to_numpy(got)
    assert np.array_equal(rp, want[0]) and np.array_equal(e, want[1]) and np.array_equal(c, want[2])


# one pair: a single range; several; odd n and the second pair word (n > 8);
# more rows than a step of 512 threads; one row, one partner; wide cells with
# 512-thread workgroups
@pytest.mark.parametrize("n,d,ta,tb", [
    (2, 20, 100, 100), (3, 9, 200, 201), (4, 6, 200, 200), (7, 3, 65, 67), (9, 3, 210, 130), (13, 2, 100, 101),
    (16, 2, 150, 150), (5, 8, 1200, 7), (5, 8, 7, 1200), (2, 60, 1, 1800), (2, 60, 1800, 3), (10, 5, 2500, 1100),
])
def test_one_pair(n, d, ta, tb):
    rng = W.rng_for(71000 + 100 * n + d)
    a, b = _poly(rng, n, d, ta), _poly(rng, n, d, tb)
    got = ph.mul(_batch([a], n, d), _batch([b], n, d))
    e, c = oracle.mul(*a, *b)
    _same(got, (np.array([0, len(c)]), e, c))


def test_repeated_monomials_zeros_and_tolerance():
    """Equal monomials in both operands keep storage order; exact
    cancellations, a tolerance, infinities and NaN as the definition has them."""
    rng = W.rng_for(72001)
    n, d = 4, 3
    a, b = _poly(rng, n, d, 160, repeats=True), _poly(rng, n, d, 150, repeats=True)
    ai = (a[0], np.round(a[1] * 3))
    bi = (b[0], np.round(b[1] * 3))
    for x, y, tol in ((a, b, 0.0), (ai, bi, 0.0), (a, b, 0.75)):
        e, c = oracle.mul(*x, *y, tol)
        _same(ph.mul(_batch([x], n, d), _batch([y], n, d), tol), (np.array([0, len(c)]), e, c))
    bad = a[1].copy()
    bad[3], bad[40] = np.inf, np.nan
    e, c = oracle.mul(a[0], bad, *b)
    rp, ge, gc = ph.batch_to_numpy(ph.mul(_batch([(a[0], bad)], n, d), _batch([b], n, d)))
    assert np.array_equal(ge, e) and np.array_equal(gc, c, equal_nan=True)


def test_batch_with_empty_and_ragged_entries():
    rng = W.rng_for(72002)
    n, d = 5, 3
    sizes = [(0, 5), (5, 0), (1, 1), (56, 56), (3, 40), (40, 3), (17, 29), (56, 1)] * 6
    pa = [_poly(rng, n, d, s) for s, _ in sizes]
    pb = [_poly(rng, n, d, s) for _, s in sizes]
    want = [oracle.mul(*x, *y) if len(x[1]) and len(y[1]) else (np.zeros((0, n), np.uint8), np.zeros(0))
            for x, y in zip(pa, pb)]
    got = ph.mul(_batch(pa, n, d), _batch(pb, n, d))
    _same(got, W.csr_from_list(want, n))


@pytest.mark.parametrize("I,K,J", [(1, 1, 1), (2, 3, 2), (1, 5, 4), (4, 1, 3)])
def test_matrix_products(I, K, J):
    rng = W.rng_for(73000 + 100 * I + 10 * K + J)
    n, d = 4, 4
    pa = [_poly(rng, n, d, int(t)) for t in rng.integers(0, 70, I * K)]
    pb = [_poly(rng, n, d, int(t)) for t in rng.integers(30, 70, K * J)]
    pa[0] = _poly(rng, n, d, 70)
    a, b = _batch(pa, n, d), _batch(pb, n, d)
    want = oracle.mtimes(*W.csr_from_list(pa, n), *W.csr_from_list(pb, n), I, K, J)
    _same(ph.mtimes(a, b, I, K, J), want)


def test_declared_bounds_above_the_data_and_below_it():
    """A generous max_exp changes the keys, not the result; an exponent above
    the declared bound is the device status it was."""
    rng = W.rng_for(72003)
    n, d = 4, 6
    a, b = _poly(rng, n, d, 150), _poly(rng, n, d, 150)
    e, c = oracle.mul(*a, *b)
    _same(ph.mul(_batch([a], n, 60), _batch([b], n, 100)), (np.array([0, len(c)]), e, c))
    low = int(a[0].max()) - 1
    with pytest.raises(ph.PolyError):
        ph.mul(_batch([a], n, low), _batch([b], n, d))


def test_general_route_agrees():
    """The route without degrees (finish=False, as under capture) gives the same bits."""
    rng = W.rng_for(72004)
    n, d = 6, 4
    a, b = _batch([_poly(rng, n, d, 200)], n, d), _batch([_poly(rng, n, d, 190)], n, d)
    x = ph.mul(a, b)
    y = ph.mul(a, b, finish=False)
    torch.cuda.synchronize()
    rp = y.row_ptr.cpu().numpy()
    T = int(rp[-1])
    assert np.array_equal(rp, x.row_ptr_host)
    assert torch.equal(y.exps[:T], x.exps) and torch.equal(y.coefs[:T], x.coefs)


def _capped(rng, n, d, cap, t):
    """t distinct monomials of degree <= d with exponents <= cap; the largest
    exponent and the largest degree are both met."""
    e = np.zeros((0, n), np.uint8)
    while len(e) < t:
        u = np.zeros((4 * t, n), np.uint8)
        for r in u:
            for i in rng.integers(0, n, rng.integers(0, d + 1)):
                r[i] = min(r[i] + 1, cap)
        e = np.unique(np.concatenate([e, u]), axis=0)
    e = e[rng.permutation(len(e))[:t]]
    top = np.zeros(n, np.uint8)
    for k in range(d):
        top[k // cap] += 1
    if not (e == top).all(axis=1).any():
        e[0] = top
    return e, rng.standard_normal(t)


# Exponents bounded below the degree: a product key's radix, amax + bmax + 1,
# is then at most the product's degree, and a range may begin at a monomial
# that no product can be (keys as large as 3^16, 4^13, 5^9, 2^16).
@pytest.mark.parametrize("n,d,amax,bmax,t", [
    (7, 3, 1, 1, 64), (8, 3, 1, 1, 93), (10, 3, 1, 1, 150), (16, 3, 1, 1, 400), (11, 4, 1, 1, 350),
    (8, 4, 1, 2, 150), (9, 3, 2, 1, 150), (5, 6, 2, 2, 130), (6, 5, 3, 1, 180), (13, 3, 1, 2, 300), (6, 4, 1, 0, 64),
])
def test_exponent_bounds_below_the_degree(n, d, amax, bmax, t):
    rng = W.rng_for(74000 + 1000 * n + 100 * d + 10 * amax + bmax)
    a = _capped(rng, n, d, amax, t if amax > 1 else min(t, sum(math.comb(n, k) for k in range(d + 1))))
    if bmax:
        b = _capped(rng, n, min(d, n * bmax), bmax, t if bmax > 1 else min(t, sum(math.comb(n, k) for k in range(d + 1))))
    else:
        b = np.zeros((t, n), np.uint8), rng.standard_normal(t)
    e, c = oracle.mul(*a, *b)
    _same(ph.mul(_batch([a], n, amax), _batch([b], n, bmax)), (np.array([0, len(c)]), e, c))


def test_inferred_exponent_bounds():
    """max_exp left to batch_from_numpy is the largest exponent: all 93
    multilinear monomials of degree <= 3 in 8 variables, squared, as one pair,
    as a batch and as a matrix product."""
    rng = W.rng_for(74001)
    n = 8
    e = np.array([[1 if i in s else 0 for i in range(n)] for k in range(4) for s in itertools.combinations(range(n), k)],
                 np.uint8)
    polys = [(e, rng.standard_normal(len(e))) for _ in range(6)]
    rp, ee, cc = W.csr_from_list(polys, n)
    one = [ph.batch_from_numpy([0, len(e)], *p, n=n) for p in polys]
    x, c = oracle.mul(*polys[0], *polys[1])
    _same(ph.mul(one[0], one[1]), (np.array([0, len(c)]), x, c))
    many = ph.batch_from_numpy(rp, ee, cc, n=n)
    assert many.max_exp == 1
    _same(ph.mul(many, many), W.csr_from_list([oracle.mul(*p, *p) for p in polys], n))
    _same(ph.mtimes(many, many, 2, 3, 2), oracle.mtimes(rp, ee, cc, rp, ee, cc, 2, 3, 2))


@pytest.mark.parametrize("own", [False, True])
def test_no_memory_for_the_staged_cells(monkeypatch, own):
    """Cells take more memory than the general route's raw products where the
    product is sparse: without it the call takes the general route, in a
    workspace of its own or the caller's."""
    rng = W.rng_for(75001)
    n, d, P, t = 8, 4, 400, 45
    a, b = (_batch([_poly(rng, n, d, t) for _ in range(P)], n, d) for _ in range(2))
    want = ph.mul(a, b)
    need, raw = ph.mul_workspace(a, b)
    asked = []
    make = ph._workspace

    def limited(nbytes, device):
        asked.append(nbytes)
        if nbytes > need:
            raise torch.OutOfMemoryError("no memory")
        return make(nbytes, device)

    monkeypatch.setattr(ph, "_workspace", limited)
    got = ph.mul(a, b, ws=make(need, "cuda") if own else None)
    assert max(asked) > need   # the route was tried
    assert np.array_equal(got.row_ptr_host, want.row_ptr_host)
    assert torch.equal(got.exps, want.exps) and torch.equal(got.coefs, want.coefs)
    with pytest.raises(torch.OutOfMemoryError):
        monkeypatch.setattr(ph, "_workspace", lambda nbytes, device: (_ for _ in ()).throw(torch.OutOfMemoryError()))
        ph.mul(a, b)


def test_host_offsets_beyond_the_device_s():
    """The host's offsets plan the launches, the device's say what the
    operands are: where the host's copy is only a bound, the terms past the
    device's last offset take no part."""
    rng = W.rng_for(76001)
    n, d = 6, 4
    pa, pb = [_poly(rng, n, d, t) for t in (90, 150)], [_poly(rng, n, d, t) for t in (130, 170)]
    for ta, tb in ((150, 100), (1, 170), (149, 1), (0, 170), (150, 170)):
        a, b = _batch(pa, n, d), _batch(pb, n, d)
        a.row_ptr[2] = 90 + ta
        b.row_ptr[2] = 130 + tb
        qa, qb = [pa[0], (pa[1][0][:ta], pa[1][1][:ta])], [pb[0], (pb[1][0][:tb], pb[1][1][:tb])]
        want = [oracle.mul(*x, *y) if len(x[1]) else (np.zeros((0, n), np.uint8), np.zeros(0)) for x, y in zip(qa, qb)]
        _same(ph.mul(a, b), W.csr_from_list(want, n))
