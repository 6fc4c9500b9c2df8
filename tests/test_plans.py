"""Launch plans, which the host computes from sizes alone (no GPU needed)."""
import ctypes as C
import os

import pytest

from util import binding, internal


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2603_17942_amd import build
        build.build(verbose=False)


@pytest.mark.parametrize("m,ff,full,batch", [
    (128, 14336, 0b001, 0b001), (320, 14336, 0b001, 0b001), (352, 14336, 0b010, 0b011), (400, 14336, 0b010, 0b011),
    (512, 14336, 0b010, 0b010), (640, 14336, 0b001, 0b011), (1344, 14336, 0b001, 0b011), (2112, 14336, 0b010, 0b011),
    (400, 12288, 0b010, 0b011), (560, 12288, 0b100, 0b110), (640, 12288, 0b001, 0b111), (2048, 12288, 0b010, 0b011)])
def test_gate_up_tiles(m, ff, full, batch):
    """Tiles launched for the gate/up projection (bit 0 gemm_plan's, 1: 256 x 256, 2: 192 x 320) of m rows, and of a batch of m
    block rows, of which only the device knows how many are there: one that suits two thirds of them, and one that suits all
    (640 rows: up to 512 there one round of 256 x 256, more two of the ring)."""
    tiles = internal("gate_up_tiles", C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_bool, restype=C.c_uint)
    assert tiles(m, ff, 4096, None, False) == full
    assert tiles(m, ff, 4096, None, True) == batch
    assert tiles(m, ff, 4096, 8, True) == 0b001             # results off the 16-byte alignment of the wide tiles' stores
