"""Small products whose operands are views with very long leading dimensions: the
tile class, and with it the order of the sums, follows from the shape alone, so
they give the bits of the same product of dense copies, and at 3xBF16 of packed
operands.

An operand of 100 rows of k spans 2^29 floats from a leading dimension of 5.4M on;
the offsets within a tile of 64 rows of k pass 32 bits at 2^24, those of k rows
within a step at 2^26."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


@pytest.fixture(scope="module")
def memory():
    # 10 GiB: 40 rows of the longest leading dimension and a little more
    return torch.empty(40 * (2 ** 26 + 64) + 4096, device="cuda")


@pytest.mark.parametrize("prec", [1, 2, 3])
@pytest.mark.parametrize("op,t,m,n,k,ld", [
    ("A", 0, 100, 130, 1000, 6_000_001), ("B", 1, 130, 100, 1000, 6_000_001),   # tiles of 32
    ("A", 0, 500, 700, 300, 1_100_003), ("B", 1, 700, 500, 300, 1_100_003),     # of 64
    ("A", 0, 130, 3001, 37, 2 ** 24), ("A", 0, 130, 3001, 37, 2 ** 24 + 1),
    ("B", 1, 3001, 130, 37, 2 ** 24), ("B", 1, 3001, 130, 37, 2 ** 24 + 1),
    ("A", 1, 3001, 130, 37, 2 ** 26), ("A", 1, 3001, 130, 37, 2 ** 26 + 1),
    ("B", 0, 130, 3001, 37, 2 ** 26), ("B", 0, 130, 3001, 37, 2 ** 26 + 1),
    ("A", 0, 33, 45, 100, 2 ** 26 + 1), ("B", 0, 33, 45, 35, 2 ** 26 + 1),
    ("A", 1, 1, 3, 33, 2 ** 26 + 1), ("B", 1, 3, 1, 33, 2 ** 26 + 1)])
def test_same_bits_as_dense(la, memory, prec, op, t, m, n, k, ld):
    torch.manual_seed(5 + m + n + k)
    a, b = torch.randn(m, k, device="cuda"), torch.randn(k, n, device="cuda")
    x = a if op == "A" else b
    rows, cols = x.shape[::-1] if t else x.shape
    assert rows * ld < memory.numel()
    V = memory[1:1 + rows * ld].view(rows, ld)[:, :cols]
    V = V.T if t else V
    V.copy_(x)
    dense = x.T.contiguous().T if t else x
    p = la.Precision(prec)
    for other in ((b, b.T.contiguous().T) if op == "A" else (a, a.T.contiguous().T)):
        C = la.gemm(*((V, other) if op == "A" else (other, V)), prec=p)
        assert torch.equal(C, la.gemm(*((dense, other) if op == "A" else (other, dense)), prec=p))
    if prec == 2:
        packed = la.gemm_packed(la.pack_bf16x3(a), la.pack_bf16x3(b.T.contiguous()), m, n, k)
        assert torch.equal(C, packed)
