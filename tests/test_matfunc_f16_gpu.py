"""Matrix functions whose products run on packed fp16 terms scaled row by row
(AUTO on the larger sizes) against FP64: no less accurate than the 6xBF16
products, with and without the workspace that holds the packs, and with rows and
columns of very different size.

Tolerances: normwise 2(d+1) g (the Horner bound of the matrix-function tests with
g = 1e-6), and 1.1 times the 6xBF16 run's error; small rows each to the same
bound relative to themselves."""
import numpy as np
import pytest
import torch

import la_inputs

pytestmark = pytest.mark.gpu

G = 1e-6


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def cheb64(A, c, half):
    B = A.double() / half
    t0 = torch.eye(A.shape[0], dtype=torch.float64, device="cuda")
    t1 = B
    f = c[0] * t0 + c[1] * t1
    for ck in c[2:]:
        t0, t1 = t1, 2.0 * (B @ t1) - t0
        f = f + ck * t1
    return f


def odd64(A, c):
    A = A.double()
    g = A.t() @ A
    p = torch.zeros_like(g)
    for cj in reversed(c):
        p = p @ g
        p.diagonal().add_(cj)
    return A @ p


@pytest.mark.parametrize("n,deg", [(1700, 2), (1701, 3), (2049, 6), (3000, 5)])
def test_cheb(la, n, deg):
    g = torch.Generator("cuda").manual_seed(n)
    A = torch.randn((n, n), device="cuda", generator=g) * (0.25 / n ** 0.5)
    A = (A + A.t()).contiguous()
    c = la_inputs.rng(n).standard_normal(deg + 1)
    ref = cheb64(A, c, 1.25)
    err = {}
    for name, kw in (("auto", {}), ("x6", dict(prec=la.Precision.BF16X6)),
                     ("short", dict(workspace=torch.empty(3 * 4 * n * n + 3 * 256 + 256,
                                                          dtype=torch.uint8, device="cuda")))):
        F = la.matfunc_cheb(A, -1.25, 1.25, c, **kw)
        torch.cuda.synchronize()
        err[name] = (torch.linalg.norm(F.double() - ref) / torch.linalg.norm(ref)).item()
    print(err)
    assert err["auto"] <= 2 * (deg + 1) * G and err["auto"] <= 1.1 * err["x6"]
    assert err["short"] == err["x6"]


@pytest.mark.parametrize("m,n,terms", [(2000, 3000, 4), (3000, 2000, 5), (5000, 1800, 2),
                                       (1700, 1700, 3), (40000, 1100, 3)])
def test_odd(la, m, n, terms):
    g = torch.Generator("cuda").manual_seed(m + n)
    A = torch.randn((m, n), device="cuda", generator=g) / (m ** 0.5 + n ** 0.5)
    c = [(-1.0) ** j * 0.9 / (j + 1) for j in range(terms)]
    ref = odd64(A, c)
    F = la.matfunc_odd(A, c)
    torch.cuda.synchronize()
    err = (torch.linalg.norm(F.double() - ref) / torch.linalg.norm(ref)).item()
    print(err)
    assert err <= 2 * (terms + 1) * G


def test_rows_of_very_different_size(la):
    """Rows from 2^-60 to 2^8 and a column at 2^-50: F = A p(A^T A) scales with the
    rows of A, so every row is held to the bound relative to its own norm."""
    m, n = 2500, 1800
    g = torch.Generator("cuda").manual_seed(76)
    A = torch.randn((m, n), device="cuda", generator=g) / (m ** 0.5 + n ** 0.5)
    A[:100] *= 2.0 ** -60
    A[100:200] *= 2.0 ** -30
    A[:, 7] *= 2.0 ** -50
    c = [0.9, -0.45, 0.3]
    ref = odd64(A, c)
    F = la.matfunc_odd(A, c).double()
    torch.cuda.synchronize()
    rel = torch.linalg.norm(F - ref, dim=1) / torch.linalg.norm(ref, dim=1)
    assert rel.max().item() <= 2 * 4 * G
    # scaling A by a power of two scales an F of one term and leaves its bits
    F1 = la.matfunc_odd(A, [0.5, 0.0])
    F2 = la.matfunc_odd(A * 2.0 ** 20, [0.5, 0.0])
    torch.cuda.synchronize()
    assert torch.equal(F1 * 2.0 ** 20, F2)


def test_non_finite_stay_in_their_rows(la):
    n = 1700
    g = torch.Generator("cuda").manual_seed(77)
    A = torch.randn((n, n), device="cuda", generator=g) / n ** 0.5
    A[5, 9] = float("inf")
    F = la.matfunc_cheb(A, -4.0, 4.0, [0.1, 0.2, 0.3])
    torch.cuda.synchronize()
    bad = ~torch.isfinite(F)
    assert bool(bad[5].any()) and not bool(bad[:, :].all())
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[5] = False
    cols = torch.ones(n, dtype=torch.bool, device="cuda")
    cols[9] = False
    assert not bool(bad[keep][:, cols].any())
