"""Choice of la_gemm's tile class where it depends on K.

256 x 256 and 128 x 128 tiles add in the same order, so a product that takes one
of them is bitwise the leading block of a wider product that takes the other: the
two shapes below lie on either side of the rule of la_gemm (the cost of a round of
each, restated here).  A third round of 64 x 64 tiles is taken from a certain K
on: around it every product is within |err| <= (8 + k) u |A||B| of FP64, entry by
entry, with u = 2^-23 (FP32, 6xBF16) or 2^-16 / 64 (3xBF16, whose dropped lo lo
products are random in sign), and the packed product has the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

COST = {1: (40.0, .2535, 9.5, .146), 2: (33.5, .0788, 8.3, .0575), 3: (32.5, .1207, 6.0, .0826)}


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def takes_small(m, n, k, prec):
    def tiles(t):
        return -(-m // t) * -(-n // t)
    l0, lk, s0, sk = COST[prec]
    return max(1.0, tiles(128) / 512) * (s0 + sk * k) < 0.97 * -(-tiles(256) // 256) * (l0 + lk * k)


def operands(m, n, k, ta, tb, seed=0):
    torch.manual_seed(7 + m + n + k + seed)
    A = torch.randn((k, m) if ta else (m, k), device="cuda")
    B = torch.randn((n, k) if tb else (k, n), device="cuda")
    return (A.T if ta else A), (B.T if tb else B)


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("k", [900, 1011])
def test_large_and_small_tiles_same_bits(la, prec, ta, tb, k):
    # 4096 x 4096 is one full round of large tiles; 100 rows more start a second
    m, n, more = 4096, 4096, 100
    assert not takes_small(m, n, k, prec) and takes_small(m + more, n, k, prec)
    a, b = operands(m + more, n, k, ta, tb)
    wide = la.gemm(a, b, prec=la.Precision(prec))
    C = la.gemm(a[:m], b, prec=la.Precision(prec))
    assert torch.equal(C, wide[:m])


@pytest.mark.parametrize("prec,m,n,ks", [(2, 1500, 1500, (639, 640)), (3, 3000, 700, (319, 320)),
                                         (1, 1450, 1450, (327, 328, 346, 399, 400)),
                                         (1, 2100, 2100, (255, 256)), (2, 200, 9000, (64, 639, 640))])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1)])
def test_third_round(la, prec, m, n, ks, ta, tb):
    for k in ks:
        a, b = operands(m, n, k, ta, tb)
        C = la.gemm(a, b, prec=la.Precision(prec))
        want = a.double() @ b.double()
        u = 2.0 ** (-22 if prec == 2 else -23)
        bound = (8 + k) * u * (a.double().abs() @ b.double().abs())
        assert torch.all((C.double() - want).abs() <= bound)
        if prec == 2:
            D = la.gemm_packed(la.pack_bf16x3(a), la.pack_bf16x3(b.T), m, n, k)
            assert torch.equal(C, D)


@pytest.mark.parametrize("m,n,k", [(4096, 2048, 256), (100, 33000, 300), (32513, 7, 256)])
def test_workspace_is_asked_for(la, m, n, k):
    # 3xBF16 with at least 128 tiles of 256 x 256, also where a side is below 256
    a, b = operands(m, n, k, 0, 0)
    short = torch.empty(la.gemm_workspace_size(m, n, k) - 1, dtype=torch.uint8, device="cuda")
    assert short.data_ptr() % 256 == 0
    with pytest.raises(la.LAError) as e:
        la.gemm_ws(a, b, workspace=short)
    assert e.value.status == la.Status.OUT_OF_MEMORY
    assert torch.equal(la.gemm_ws(a, b), la.gemm(a, b))
