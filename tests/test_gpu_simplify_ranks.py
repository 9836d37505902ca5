"""simplify of large batches of low degree (sorted by monomial rank in LDS), bit
for bit against the general path, which finish=False takes, and the oracle: at
the polynomial sizes where the workgroup changes, with runs longer than a round,
one monomial only, rows that are no whole words, and just past the sizes,
degrees and variables that the rank path takes."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2604_06575_amd as ph

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 64, 65, 255, 256, 257, 1023, 0, 1024, 1025, 8191, 8192, 8193, 20479, 20480, 3]


def _batch(rng, n, d, sizes):
    T = sum(sizes)
    f = rng.integers(0, n + 1, size=(T, d))
    e = np.zeros((T, n + 1), np.uint8)
    np.add.at(e, (np.arange(T)[:, None], f), 1)
    c = rng.integers(-3, 4, T) * rng.choice([1.0, 0.1, 1e16, -0.0], T)
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64), np.ascontiguousarray(e[:, :n]), c


@pytest.mark.parametrize("n,d,sizes", [
    (20, 6, EDGES), (7, 3, EDGES), (2, 3, EDGES), (3, 0, EDGES), (1, 40, EDGES), (9, 12, EDGES), (128, 3, EDGES),
    (20, 6, [20481] + EDGES), (129, 2, EDGES), (24, 9, EDGES), (5, 60, EDGES), (20, 6, [30] * 3000),
])
def test_simplify_ranks(n, d, sizes):
    rng = np.random.default_rng(1000 * n + d + len(sizes))
    rp, e, c = _batch(rng, n, d, sizes)
    b = ph.batch_from_numpy(rp, e, c)
    for tol in (0.0, 0.25):
        got = ph.simplify(b, tol)
        g = ph.simplify(b, tol, finish=False)
        torch.cuda.synchronize()
        assert torch.equal(got.row_ptr, g.row_ptr)
        T = got.nterms
        assert torch.equal(got.exps, g.exps[:T])
        assert torch.equal(got.coefs.view(torch.int64), g.coefs[:T].view(torch.int64))
    if n in (2, 7):
        orp, oe, oc = oracle.simplify_batch(rp, e, c, 0.25, n=n)
        grp, ge, gc = ph.batch_to_numpy(got)
        assert np.array_equal(grp, orp) and np.array_equal(ge, oe)
        assert np.array_equal(gc.view(np.uint64), np.asarray(oc).view(np.uint64))


def test_capacity_and_exponent_status():
    rng = np.random.default_rng(5)
    rp, e, c = _batch(rng, 6, 4, [40000 // 2] * 4)
    b = ph.batch_from_numpy(rp, e, np.abs(c) + 1)
    small = ph.batch_from_numpy(np.zeros(5, np.int64), np.zeros((7, 6), np.uint8), np.zeros(7), n=6, max_exp=4)
    with pytest.raises(ph.PolyError):
        ph.simplify(b, out=small)
    with pytest.raises(ph.PolyError):
        ph.simplify(ph.batch_from_numpy(rp, e, c, n=6, max_exp=3))


# rows that begin and end within words, in one block and in many; the largest
# degree in the last row, the first, and one that ends at a block's edge
@pytest.mark.parametrize("n,T", [(3, 2048), (5, 2049), (7, 30000), (21, 9000), (33, 4000), (61, 2500), (127, 2100), (127, 9001), (128, 5000)])
def test_degree_is_read_whole(n, T):
    rng = np.random.default_rng(n + T)
    e = np.zeros((T, n), np.uint8)
    e[np.arange(T), rng.integers(0, n, T)] = 1
    for t, i in ((T - 1, n - 1), (0, 0), (1023 if T > 1023 else T // 2, n // 2)):
        x = e.copy()
        x[t] = 0
        x[t, i] = 4
        b = ph.batch_from_numpy([0, T // 2, T], x, np.ones(T), n=n)
        words = torch.zeros(2, dtype=torch.int64, pin_memory=True)
        scratch = torch.zeros(16, dtype=torch.uint8, device="cuda")
        c = b.csr()
        assert ph.lib().simplify_degree(ctypes.byref(c), scratch.data_ptr(), words.data_ptr(),
                                        torch.cuda.current_stream().cuda_stream) == 0
        assert int(words[0]) == 4


def test_host_offsets_beyond_the_device_s():
    rng = np.random.default_rng(77)
    sizes = [3000, 20, 400, 9000]
    rp, e, c = _batch(rng, 7, 4, sizes)
    for last in (0, 1, 300, 8999):
        b = ph.batch_from_numpy(rp, e, c)
        b.row_ptr[4] = int(rp[3]) + last
        T = int(rp[3]) + last
        drp = np.append(rp[:4], T)
        orp, oe, oc = oracle.simplify_batch(drp, e[:T], c[:T], 0.0, n=7)
        grp, ge, gc = ph.batch_to_numpy(ph.simplify(b))
        assert np.array_equal(grp, orp) and np.array_equal(ge, oe)
        assert np.array_equal(gc.view(np.uint64), np.asarray(oc).view(np.uint64))
