"""The workspace holds a partial sum for every workgroup of every reduction: the
tiles of the residual passes over any box of the mesh, and the box kernels'."""
from __future__ import annotations

import ctypes
import itertools

import pytest

import paper_1709_04703_amd as P


class Box(ctypes.Structure):
    _fields_ = [("lo", ctypes.c_int * 3), ("hi", ctypes.c_int * 3)]


def reserved(n):
    fn = P.library()._ZN4sdpm16reduction_blocksEi        # int64_t reduction_blocks(int)
    fn.restype = ctypes.c_int64
    return fn(n)


def tiles(lo, hi):
    fn = P.library()._ZN4sdpm15residual_blocksERKNS_3BoxE   # int residual_blocks(const Box&)
    return fn(ctypes.byref(Box((ctypes.c_int * 3)(*lo), (ctypes.c_int * 3)(*hi))))


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024, 2048])
def test_partials_of_every_box(n):
    cells = -(-n // 64) * -(-n // 4) * -(-n // 8)        # box kernels: 64 x 4 x 8 cells
    assert reserved(n) >= cells
    # faces at, just inside and well inside the mesh's; the extents count
    lows = sorted({0, 1, 2, 3, 5, n // 4 + 1, n // 2 - 1})
    spans = sorted({1, 2, 3, 7, n // 4, n // 2, n - 7, n - 4, n - 3, n - 2, n - 1, n} - {0, -1, -3})
    xs = [(lo, lo + s - 1) for lo, s in itertools.product(lows, spans) if lo + s <= n]
    for x in xs:
        for y, z in itertools.product(spans, spans):
            assert tiles((x[0], 0, 0), (x[1], y - 1, z - 1)) <= reserved(n)
