"""Device bytes that callers reserve (no GPU): a workspace or a server arena of the
size that was enough before stays enough."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2010_10272_amd", "libhgref.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    import torch  # noqa: F401  (same HIP runtime the product binds to)
    return ctypes.CDLL(LIB)


# n, m, P, k_max -> hg_workspace_size, hg_request_bytes (5 rounds, vertex weights)
KEPT = [((1, 1, 1, 2), 79360, 82688),
        ((10_000, 10_000, 40_000, 2), 747008, 1599232),
        ((1_000_000, 1_000_000, 10_000_000, 64), 142629632, 551631616),
        ((4_000_000, 4_200_000, 56_500_000, 16), 765653760, 1672055552)]


@pytest.mark.parametrize("sizes,workspace,request_bytes", KEPT)
def test_reserved_sizes_do_not_grow(lib, sizes, workspace, request_bytes):
    i32, i64 = ctypes.c_int32, ctypes.c_int64
    lib.hg_workspace_size.argtypes = [i32, i32, i64, i32]
    lib.hg_request_bytes.argtypes = [i32, i32, i64, i32, i32, i32, i32]
    lib.hg_workspace_size.restype = lib.hg_request_bytes.restype = ctypes.c_size_t
    assert 0 < lib.hg_workspace_size(*sizes) <= workspace
    assert 0 < lib.hg_request_bytes(*sizes, 5, 1, 0) <= request_bytes
