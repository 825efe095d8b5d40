"""The direct GEMM kernels (operands straight into MFMA fragments, the waves of a
workgroup splitting K) against the FP64 oracle, at the edges of their tiles and
steps: every layout pair and precision, odd sizes, partial 16-k steps, views at
an odd offset and leading dimension, one row or column, alpha/beta, and the
Gram and partial-sum paths through la_polar and la_inverse sizes around the
tile-class borders.

Tolerances: the normwise 1e-6 of the GEMM tests (for 3xBF16 max(1e-6,
2^-16 / sqrt(K)), from its dropped lo*lo products), and integer inputs exact."""
import numpy as np
import pytest
import torch

import la_inputs
import oracle

pytestmark = pytest.mark.gpu

PRECS = ["FP32", "BF16X3", "BF16X6"]


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def operand(shape, trans, seed, pad, integer=False):
    """op(X) of the given shape as a device view: transposed or not, inside a
    larger buffer at an odd offset when pad is odd."""
    r, c = shape[::-1] if trans else shape
    g = la_inputs.integer_matrix if integer else la_inputs.gaussian
    big = g((r + 1, c + pad), seed)
    v = torch.from_numpy(big).to("cuda")[1:, pad:] if pad else torch.from_numpy(big).to("cuda")[1:]
    x = big[1:, pad:]
    return (v.T, x.T) if trans else (v, x)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("mnk", [(32, 32, 16), (33, 31, 17), (1, 2, 15), (2, 1, 40), (63, 65, 127),
                                 (64, 64, 128), (545, 513, 130), (1025, 577, 65), (130, 3, 700)])
def test_edges_against_oracle(la, prec, ta, tb, mnk):
    m, n, k = mnk
    for pad, integer in ((0, False), (3, False), (1, True)):
        Av, A = operand((m, k), ta, 1000 + m, pad, integer)
        Bv, B = operand((k, n), tb, 2000 + n, pad, integer)
        C0 = la_inputs.integer_matrix((m, n), 3000) if integer else la_inputs.gaussian((m, n), 3000)
        for alpha, beta in ((1.0, 0.0), (2.0, -1.0)):
            C = torch.from_numpy(C0).to("cuda") if beta else torch.full((m, n), float("nan"),
                                                                        device="cuda")
            la.gemm(Av, Bv, C, alpha=alpha, beta=beta, prec=la.Precision[prec])
            torch.cuda.synchronize()
            ref = alpha * oracle.gemm(np.ascontiguousarray(A), np.ascontiguousarray(B))
            if beta:
                ref = ref + beta * C0.astype(np.float64)
            got = C.cpu().numpy().astype(np.float64)
            if integer:
                assert np.array_equal(got, ref), (pad, alpha, beta)
                continue
            nrm = alpha * np.linalg.norm(A) * np.linalg.norm(B) + abs(beta) * np.linalg.norm(C0)
            tol = max(1e-6, 2.0 ** -16 / np.sqrt(k)) if prec == "BF16X3" else 1e-6
            assert np.linalg.norm(got - ref) <= tol * nrm, (pad, alpha, beta)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("mnk", [(2049, 2050, 33), (2100, 2177, 100), (129, 20000, 70),
                                 (257, 33000, 48), (3001, 2999, 40)])
def test_staged_tiles_at_the_edges(la, prec, mnk):
    """Staged tiles whose last row and column of tiles are moved back inside the
    matrix, with odd leading dimensions and offsets and C updated in place
    (beta): integers, so exact, elements shared by two tiles counted once."""
    m, n, k = mnk
    for ta, tb in ((False, False), (True, True)):
        Av, A = operand((m, k), ta, 61, 1, True)
        Bv, B = operand((k, n), tb, 62, 3, True)
        C0 = la_inputs.integer_matrix((m, n), 63)
        C = torch.from_numpy(C0).to("cuda")
        la.gemm(Av, Bv, C, alpha=1.0, beta=-2.0, prec=la.Precision[prec])
        ref = (torch.from_numpy(A.copy()).to("cuda").double() @
               torch.from_numpy(B.copy()).to("cuda").double()) - 2.0 * torch.from_numpy(C0).to("cuda")
        torch.cuda.synchronize()
        assert torch.equal(C.double(), ref)


@pytest.mark.parametrize("mnk", [(96, 70, 50), (513, 512, 257), (1100, 1000, 333)])
def test_packed_operands_bitwise(la, mnk):
    """la_gemm_packed adds as la_gemm does in both direct classes."""
    m, n, k = mnk
    A = torch.from_numpy(la_inputs.gaussian((m, k), 41)).to("cuda")
    B = torch.from_numpy(la_inputs.gaussian((k, n), 42)).to("cuda")
    C0 = la.gemm(A, B, alpha=1.5, prec=la.Precision.BF16X3)
    C1 = la.gemm_packed(la.pack_bf16x3(A), la.pack_bf16x3(B.T), m, n, k, alpha=1.5)
    torch.cuda.synchronize()
    assert torch.equal(C0, C1)


@pytest.mark.parametrize("n", [31, 33, 511, 705, 1000])
def test_step_norm_and_symmetry(la, n):
    """The Gram and the step-norm partials of the direct classes: H exactly
    symmetric, the last step norm against the FP64 norm of an extra step."""
    case = la_inputs.polar_case(n, n, 1e-1, seeds=(51, 52, 53))
    A = torch.from_numpy(case.A32).to("cuda")
    U, H, info = la.polar(A)
    U1, _, i1 = la.polar(A, max_iter=info["iters_ns"] - 1, stagnation=False,
                         raise_not_converged=False)
    torch.cuda.synchronize()
    assert torch.equal(H, H.t())
    want = torch.linalg.norm(U.double() - U1.double()).item()
    assert info["iters_ns"] == i1["iters_ns"] + 1
    assert abs(info["last_delta"] - want) <= 1e-9 * want + 1e-12
