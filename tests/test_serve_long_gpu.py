"""Served requests so long that their tiles of 32 or 64 rows would pass the tick's tile
items, and ones just short of it, are taken.  The columns of A have disjoint rows, so P is
diagonal and every step scales them: those of U have the directions of A's, to the polar
tolerance 1e-5.  (Their lengths are another matter: a served Gram is one sum over all
rows, whose rounding grows with their number.)"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("m,n", [(12_400_000, 1), (12_600_000, 1), (25_200_000, 2)])
def test_long_request(m, n):
    import paper_2112_09017_amd as la
    rng = np.random.default_rng(m)
    a = rng.standard_normal(m).astype(np.float32)
    A = np.zeros((m, n), np.float32)
    for j in range(n):
        A[j::n, j] = a[j::n]
    with la.Server(1 << 30) as srv:
        rid = srv.submit(A)
        r, t0 = None, time.time()
        while r is None and time.time() - t0 < 60.0:
            r = srv.poll(rid)
            time.sleep(0.01)
    st, U, H, info = r
    assert st == la.Status.OK
    for j in range(n):
        u, a = U[:, j].astype(np.float64), A[:, j].astype(np.float64)
        assert np.linalg.norm(u / np.linalg.norm(u) - a / np.linalg.norm(a)) <= TOL
    assert np.isfinite(H).all()
