"""Products with 256 x 256 tiles' worth of output and a short K, which run on 128 x 128
tiles where those rounds are cheaper: the same sums in the same order, so a product
is bitwise the first rows and columns' worth of a larger one that keeps the other
class, and close to FP64: |err| <= (k + 8) u |A||B| entry by entry at 3xBF16 with
u = 2^-16 (its dropped lo lo products) and 2^-23 at the others."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(3392, 4672, 91), (2817, 3001, 33), (4100, 2600, 1)])
def test_short_k(la, m, n, k, ta, tb, prec):
    torch.manual_seed(7 + m + k)
    A = torch.randn((k, m) if ta else (m, k), device="cuda")
    B = torch.randn((n, k) if tb else (k, n), device="cuda")
    a, b = (A.T if ta else A), (B.T if tb else B)
    C = la.gemm(a, b, prec=la.Precision(prec))
    ws = torch.empty(la.lib().la_gemm_workspace_size(m, n, k) + 256, dtype=torch.uint8,
                     device="cuda")
    D = la.gemm_ws(a, b, prec=la.Precision(prec), workspace=ws)
    assert torch.equal(C, D)
    want = a.double() @ b.double()
    u = 2.0 ** (-16 if prec == 2 else -23)
    bound = (8 + (k if prec != 2 else k / 64)) * u * (a.double().abs() @ b.double().abs())
    assert torch.all((C.double() - want).abs() <= bound)
