"""la_polar's FP32-level phases on two scaled fp16 terms (AUTO from n = 192)
against the FP64 oracle, around the size where they begin and at the edges of
their tiles, and over the range of ||A||_F in which H takes them.

Tolerances are the polar's: residual, orthogonality and H within 1e-5, U within
the first-order perturbation bound of that input error; AUTO's U and H may be no
further from the oracle than 1.1 times the explicit 6xBF16 phases' (the two
differ in rounding only)."""
import numpy as np
import pytest
import torch

import la_inputs
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5
X6 = dict(prec_precond=3, prec_h=3)


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def run(la, A32, **opts):
    U, H, info = la.polar(torch.from_numpy(np.ascontiguousarray(A32)).to("cuda"), **opts)
    torch.cuda.synchronize()
    return U.cpu().numpy().astype(np.float64), H.cpu().numpy().astype(np.float64), info


@pytest.mark.parametrize("shape", [(191, 191), (192, 192), (193, 193), (257, 255), (300, 192),
                                   (1500, 200), (640, 512)])
def test_against_oracle_and_x6(la, shape):
    m, n = shape
    case = la_inputs.polar_case(m, n, 1e-2, seeds=(900 + m, 901 + n, 902))
    A = case.A32.astype(np.float64)
    nA = np.linalg.norm(A)
    Uo, Ho, _ = oracle.polar(A)
    s = np.sort(case.s)
    err = {}
    for name, o in (("auto", {}), ("x6", X6)):
        U, H, info = run(la, case.A32, **o)
        assert info["prec_precond"] == 3 and info["prec_h"] == 3
        assert np.linalg.norm(U.T @ U - np.eye(n)) / np.sqrt(n) <= TOL
        assert np.linalg.norm(A - U @ H) / nA <= TOL
        assert np.array_equal(H, H.T)
        err[name] = (np.linalg.norm(U - Uo), np.linalg.norm(H - Ho) / nA)
    print(shape, err)
    assert err["auto"][0] <= 2 * TOL * nA / (s[0] + s[1])
    assert err["auto"][1] <= TOL
    for a, x in zip(err["auto"], err["x6"]):
        assert a <= 1.1 * x


def test_any_norm_of_a(la):
    """U does not depend on the scale of A; H scales with it: bit for bit while
    both norms take the fp16 terms (2^-60 < ||A||_F < 2^60), within the
    tolerance beyond."""
    case = la_inputs.polar_case(240, 208, 1e-3, seeds=(911, 912, 913))
    U, H, _ = run(la, case.A32)
    nH = np.linalg.norm(H)
    for k in (-80, -45, 45, 80):
        Uk, Hk, _ = run(la, case.A32 * np.float32(2.0 ** k))
        assert np.array_equal(Uk, U)
        if abs(k) == 45:
            assert np.array_equal(Hk, H * 2.0 ** k)
        assert np.linalg.norm(Hk * 2.0 ** -k - H) <= TOL * nH


def test_columns_of_very_different_size(la):
    """Columns down to 2^-14 of the largest: entries far below the fp16 range's
    top keep the residual within the tolerance."""
    g = la_inputs.rng(914)
    A = g.standard_normal((400, 220)) * 2.0 ** -np.linspace(0, 14, 220)[None, :]
    A32 = A.astype(np.float32)
    U, H, _ = run(la, A32)
    A = A32.astype(np.float64)
    assert np.linalg.norm(U.T @ U - np.eye(220)) / np.sqrt(220) <= TOL
    assert np.linalg.norm(A - U @ H) / np.linalg.norm(A) <= TOL
