"""Tile and split rules of the GEMM plan, on the host: each row is a size at
which both sides were timed, and the side that was faster (a split's reduction
counted).  The plan functions are C++ symbols of the library; calling them
needs no GPU."""
import ctypes

import pytest

from paper_2608_27384_amd import flashvla as fvb


class Plan(ctypes.Structure):
    _fields_ = [("tile", ctypes.c_int), ("ks", ctypes.c_int), ("tiles", ctypes.c_int),
                ("dma", ctypes.c_bool), ("ws_floats", ctypes.c_size_t)]


def _plan(M, N, K, bf16=True, reduce_fused=False):
    f = getattr(fvb.lib(), "_ZN2fv9plan_gemmEiiibb")
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 3 + [ctypes.c_bool] * 2
    return f(M, N, K, bf16, reduce_fused)


# (rows, columns, k): split or not, where the reduction is a kernel of its own
@pytest.mark.parametrize("M,N,K,split", [
    (80, 384, 1920, True), (400, 384, 1920, True), (80, 512, 1792, True), (128, 1024, 1920, True),
    (80, 384, 1536, True), (192, 2560, 1024, False), (256, 2560, 1920, False),
    (320, 2048, 1920, False), (384, 1280, 768, False), (80, 512, 1024, False),
    (256, 2560, 2048, False)])
def test_split_where_it_was_faster(M, N, K, split):
    p = _plan(M, N, K)
    assert (p.ks > 1) == split
    assert p.ws_floats == (p.ks * M * N if split else 0)


# (rows, columns, k, tiles of the faster tile: 64x128 or 128x128)
@pytest.mark.parametrize("M,N,K,tiles", [
    (1155, 2560, 1024, 19 * 20), (1300, 3072, 1024, 21 * 24), (1300, 3072, 768, 21 * 24),
    (1300, 2560, 1024, 11 * 20), (1500, 2560, 1536, 12 * 20), (850, 4096, 1024, 7 * 32),
    (1000, 4096, 1024, 8 * 32), (1150, 3072, 768, 9 * 24)])
def test_tile_that_was_faster(M, N, K, tiles):
    assert _plan(M, N, K).tiles == tiles


def test_long_products_leave_the_direct_to_lds_kernel():
    for M in (66, 5000):
        for rf in (False, True):
            assert _plan(M, 1024, (1 << 22) - 64, reduce_fused=rf).dma
            assert not _plan(M, 1024, 1 << 22, reduce_fused=rf).dma
