"""The packed-operand kernel's three tile sizes and the products of the small
class on packed operands: bit for bit the unpacked kernels' results, whichever
tile the shape takes and whether or not the workspace has room for the packs."""
import ctypes

import pytest
import torch

import la_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


# 256: 4096^2 (256 tiles); 192: 3000^2 (256 of 192 x 192), a last tile reaching past
# the padded rows (3072 = 12 x 256 = 16 x 192; 3328 = 13 x 256: 18 tiles end at
# 3456); 128: 4700^2, and the small class
@pytest.mark.parametrize("mnk", [(4096, 4096, 70), (3000, 3001, 260), (3072, 3072, 33),
                                 (3328, 2816, 50), (4700, 4690, 48), (1800, 2000, 300),
                                 (300, 9000, 100), (2817, 2815, 17)])
def test_gemm_packed_tiles_bitwise(la, mnk):
    m, n, k = mnk
    A = torch.from_numpy(la_inputs.gaussian((m, k), 71)).to("cuda")
    B = torch.from_numpy(la_inputs.gaussian((k, n), 72)).to("cuda")
    C0 = torch.from_numpy(la_inputs.gaussian((m, n), 73)).to("cuda")
    C1 = C0.clone()
    la.gemm(A, B, C0, alpha=0.5, beta=-1.0, prec=la.Precision.BF16X3)
    la.gemm_packed(la.pack_bf16x3(A), la.pack_bf16x3(B.T), m, n, k, C1, alpha=0.5, beta=-1.0)
    torch.cuda.synchronize()
    assert torch.equal(C0, C1)


def raw_polar(la, A, ws_bytes):
    """la_polar through the C ABI with a workspace of exactly ws_bytes."""
    from paper_2112_09017_amd._binding import PolarInfo, context
    m, n = A.shape
    U = torch.empty_like(A)
    H = torch.empty((n, n), device="cuda")
    ws = torch.empty(ws_bytes + 256, dtype=torch.uint8, device="cuda")
    p = (ws.data_ptr() + 255) & ~255
    info = PolarInfo()
    st = la.lib().la_polar(context(0), m, n, A.data_ptr(), n, U.data_ptr(), n, H.data_ptr(), n, p,
                           ws_bytes, None, ctypes.byref(info), None)
    torch.cuda.synchronize()
    return st, U, H, info.as_dict()


@pytest.mark.parametrize("shape", [(1664, 1664), (1701, 1633), (4100, 1300), (2200, 1900)])
def test_polar_with_and_without_room(la, shape):
    m, n = shape
    A = torch.randn((m, n), device="cuda", generator=torch.Generator("cuda").manual_seed(74))
    A = A / m ** 0.5 + 2.0 * torch.eye(m, n, device="cuda")
    full = la.polar_workspace_size(m, n)
    pk = max(int(la.lib().la_pack_size(m, n)) + int(la.lib().la_pack_size(n, n)) + 512,
             int(la.lib().la_pack_size(n, m)) + 256)
    a = raw_polar(la, A, full)
    b = raw_polar(la, A, full - pk // 2)
    assert a[0] == 0 and b[0] == 0
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2]) and a[3] == b[3]
    U = a[1].double()
    G = U.t() @ U
    G.diagonal().sub_(1.0)
    assert torch.linalg.norm(G).item() / n ** 0.5 <= 1e-5
    r = torch.linalg.norm(A.double() - U @ a[2].double()) / torch.linalg.norm(A.double())
    assert r.item() <= 1e-5


@pytest.mark.parametrize("shape", [(1700, 1700), (2000, 1500), (1500, 2100), (3000, 3000)])
def test_inverse_small_class_packs(la, shape):
    """Residual of the AUTO inverse on packed operands against all-FP32 MFMA's."""
    n, m = shape
    g = torch.Generator("cuda").manual_seed(75)
    A = torch.randn((n, m), device="cuda", generator=g) / max(n, m) ** 0.5
    A = A + 2.0 * torch.eye(n, m, device="cuda")
    res = {}
    for name, o in (("auto", {}), ("fp32", dict(prec=1))):
        X, info = la.inverse(A, **o)
        torch.cuda.synchronize()
        P = X.double() @ A.double() if n >= m else A.double() @ X.double()
        P.diagonal().sub_(1.0)
        res[name] = torch.linalg.norm(P).item() / P.shape[0] ** 0.5
    print(res)
    assert res["auto"] <= 1.25 * res["fp32"] + 1e-7
