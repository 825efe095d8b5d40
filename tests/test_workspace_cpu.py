"""Workspaces laid out by the sizes that the calls have asked for from the beginning
are large enough (regions added since are optional): the size each call requires, read
from its refusal of a workspace of one byte, which comes before any use of a device,
is at most the size recorded here."""
import ctypes
import re

import pytest

from paper_2112_09017_amd import _binding


def required(name, *args):
    """The call with made-up addresses for its operands (None: NULL), a context and a
    workspace of one byte (WS)."""
    L = _binding.lib()
    ctx = ctypes.create_string_buffer(256)
    mem = ctypes.create_string_buffer(1024)
    ws = (ctypes.addressof(mem) + 255) & ~255
    full = [ctypes.addressof(ctx)]
    for a in args:
        full += [ws, 1] if a is WS else [a]
    assert getattr(L, name)(*full) != 0
    return int(re.search(r"workspace 1 bytes, need (\d+)", L.la_last_error().decode()).group(1))


WS = object()
A, X, H = 1 << 44, 2 << 44, 3 << 44


@pytest.mark.parametrize("m,n,panel,q,size", [
    (300, 300, 64, 1, 1056256), (2000, 2000, 32, 0, 2087424), (6144, 4096, 64, 1, 212148480),
    (16384, 16384, 64, 0, 102678784), (4000, 3000, 128, 0, 19682816),
    (4000, 3000, 1, 1, 125946112), (20000, 640, 1, 1, 114485760), (100000, 17, 16, 1, 20551168),
    (5, 5, 128, 1, 3840)])
def test_caqr(m, n, panel, q, size):
    assert required("la_caqr", m, n, A, n, X if q else None, n, panel, WS, 0, None) <= size


@pytest.mark.parametrize("m,n,size", [
    (256, 256, 1065216), (1000, 1000, 16016640), (100000, 1, 417280), (100000, 64, 26452224),
    (100000, 100, 42056960), (1000000, 3, 12089088), (10000000, 1, 40653568)])
def test_polar(m, n, size):
    assert required("la_polar", m, n, A, n, X, n, None, n, WS, None, None, None) <= size


@pytest.mark.parametrize("n,m,size", [
    (256, 256, 532992), (1000, 1000, 8008960), (1600, 1600, 20489984), (1, 100000, 415232),
    (64, 100000, 25631232), (100000, 100, 40055040), (3, 1000000, 12071424),
    (10000000, 1, 40633856)])
def test_inverse(n, m, size):
    assert required("la_inverse", n, m, A, m, X, n, WS, None, None, None) <= size
