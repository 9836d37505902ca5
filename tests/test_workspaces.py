"""Workspace queries that must not grow past what the work needs.  Planning
runs on the host and looks at no device memory."""
import ctypes
import os

import numpy as np
import pytest

import paper_2604_06575_amd as ph

pytestmark = pytest.mark.skipif(not os.path.exists(ph.library_path()), reason="library not built")


def _csr(n, max_exp, P, T):
    rp = np.linspace(0, T, P + 1).astype(np.int64)
    c = ph.PolyCSR()
    c.nvars, c.max_exp, c.npolys, c.capacity = n, max_exp, P, T
    c.row_ptr_host = rp.ctypes.data
    c.row_ptr = c.exps = c.coefs = rp.ctypes.data
    c.keep = rp
    return c


# one long polynomial at many points, short ones that the register kernel does
# not take, few points
@pytest.mark.parametrize("n,P,T,N", [
    (20, 1, 100000, 1000000), (10, 1, 20000, 300000), (20, 10000, 100000, 100000), (100, 1, 100000, 8192), (20, 1000, 100000, 4000),
])
def test_coefficient_gradients(n, P, T, N):
    """Partial sums of one row of the terms for each chunk of points, or 256
    MB; beside them factor lists and what dX needs: n + 50 bytes for each of at
    most 4 T derivative terms and 24 for each term."""
    c = _csr(n, 4, P, T)
    ws = ctypes.c_size_t()
    assert ph.lib().poly_eval_backward_workspace(ctypes.byref(c), N, 0, 0, ctypes.byref(ws)) == 0
    chunks = -(-N // min(512, 8192 // (n + 1)))
    slices = 8 * N * n * 256
    rest = 8 * T * min(n, 8) * (n + 50) + 24 * T + 64 * (P * n + 1000)
    assert ws.value <= max(8 * T * chunks, 2**28) + rest + (slices if P > 1 else 0)


# output tiles few and many, 64 and 128 rows per workgroup
@pytest.mark.parametrize("K,P,N", [(10626, 500, 5000), (10626, 100, 300), (300, 70, 200), (46376, 4096, 8192), (5000, 1, 5000)])
def test_dense_workspace_holds_when_the_rows_change(K, P, N):
    L = ph.lib()
    old = ph.tune_get("dense_f64_rows")
    sizes = []
    try:
        for rows in (64, 128):
            ph.tune_set("dense_f64_rows", rows)
            f, b = ctypes.c_size_t(), ctypes.c_size_t()
            assert L.poly_eval_dense_workspace(20, K, P, N, 0, 5, ctypes.byref(f)) == 0
            assert L.poly_eval_dense_backward_workspace(20, K, P, N, 0, 5, ctypes.byref(b)) == 0
            sizes.append((f.value, b.value))
    finally:
        ph.tune_set("dense_f64_rows", old)
    assert sizes[0] == sizes[1]
