"""Step norms whose partials, one per tile, have no room in the workspace: the norm
reported after two steps is that of the difference of the iterates after one and two,
which a cap on the steps gives, summed in FP64 (the same floats in another order:
1e-12).  On either side of the room there is: the tiles of the small products and
their count are restated here."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def tiles(m, n, t):
    return -(-m // t) * -(-n // t)


def room(m, n, least):
    return -(-max(least, tiles(m, n, 128)) // 32) * 32 + 1024


def matrix(m, n):
    g = torch.Generator("cuda").manual_seed(m + n)
    return torch.randn(m, n, device="cuda", generator=g)


def check(delta, steps):
    want = torch.linalg.norm((steps[1].double() - steps[0].double())).item()
    assert abs(delta - want) <= 1e-12 * want


@pytest.mark.parametrize("m,n,t,fits", [(131072, 64, 64, True), (131200, 64, 64, True),
                                        (262400, 64, 64, False), (1000001, 3, 64, False),
                                        (200001, 65, 64, False), (400001, 1, 32, False)])
@pytest.mark.parametrize("prec", [2, 3])
def test_polar(la, m, n, t, fits, prec):
    assert (tiles(m, n, t) <= room(m, n, 1024)) == fits
    A = matrix(m, n)
    o = dict(prec_precond=prec, prec_ns=prec, s0=0.3, eps=1e-30, raise_not_converged=False,
             want_h=False)
    steps = [la.polar(A, max_iter=k, **o) for k in (1, 2)]
    check(steps[1][2]["last_delta"], [s[0] for s in steps])


@pytest.mark.parametrize("n,m,t,prec,fits", [(131072, 64, 64, 2, True), (150000, 64, 64, 2, False),
                                             (100, 100000, 64, 2, False),
                                             (100000, 100, 64, 3, False),
                                             (2340, 2340, 64, 1, True), (2432, 2432, 64, 1, False)])
def test_inverse(la, n, m, t, prec, fits):
    assert (tiles(m, n, t) <= room(m, n, 1)) == fits
    A = matrix(n, m)
    o = dict(prec=prec, eps=1e-30, raise_not_converged=False, literal_delta=True)
    steps = [la.inverse(A, max_iter=k, **o) for k in (1, 2)]
    check(steps[1][1]["last_delta"], [s[0] for s in steps])


@pytest.mark.parametrize("m,n", [(131072, 64), (262400, 64), (1000001, 3)])
def test_served(la, m, n):
    A = matrix(m, n).cpu().numpy()
    with la.Server(2 << 30) as srv:
        out = []
        for k in (1, 2):
            rid = srv.submit(A, s0=0.3, eps=1e-30, max_iter=k)
            r = None
            t0 = time.time()
            while r is None and time.time() - t0 < 60.0:
                r = srv.poll(rid)
                time.sleep(0.001)
            out.append(r)
        check(out[1][3]["last_delta"], [torch.from_numpy(np.asarray(r[1])) for r in out])
