"""Which tiles a layer's grouped products take: the host rule behind the forward
and backward (no GPU).  The shapes are ones whose tiles were timed against each
other; the rule must keep to the faster side of each."""
import ctypes

import pytest

import test_gpu_tiles as G
from paper_2508_19078_amd import api

ROWS = ("large", "32", "64", "128")
DW = ("large", "small")


class Plan(ctypes.Structure):
    _fields_ = [("rows", ctypes.c_int), ("dw", ctypes.c_int)]


def plan(d, I, S, ns, T, k, dtype="bf16"):
    """(row tile, weight-gradient tile) of a layer with S routed and ns shared slots."""
    f = getattr(api.lib(), "_ZN2fm9tile_planEPK9moe_layerii")   # fm::tile_plan(const moe_layer*, int, int)
    f.restype, f.argtypes = Plan, [ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    L = api.moe_layer(d, I, api.MOE_BF16 if dtype == "bf16" else api.MOE_F32, S, ns, *[None] * 6)
    p = f(ctypes.addressof(L), T, k)
    return ROWS[p.rows], DW[p.dw]


# d, I, slots, rows per slot (T = rows x slots / 4, top-4): row tile, weight gradients
TIMED = [
    ((4096, 1024, 32, 80), ("64", "small")),
    ((4096, 1024, 32, 112), ("128", "large")),
    ((4096, 1024, 32, 225), ("large", "large")),      # forward 299 us large, 336 on 128 rows; backward 836, 997
    ((2048, 1408, 64, 40), ("64", "small")),
    ((2048, 1408, 64, 100), ("128", "small")),
    ((2048, 1408, 64, 144), ("large", "small")),      # 1289 us large, 1297 to 1447 on 128 rows
    ((2048, 1408, 64, 300), ("large", "large")),
    ((4096, 1408, 128, 50), ("128", "small")),
    ((4096, 1408, 128, 150), ("large", "large")),     # 4276 us large, 4554 on 128 rows
    ((3072, 1536, 24, 72), ("64", "small")),
    ((3072, 1536, 24, 176), ("large", "large")),
    ((4096, 688, 16, 128), ("64", "small")),
    ((4096, 688, 16, 208), ("128", "small")),
    ((4096, 688, 16, 304), ("large", "large")),
    ((1024, 2816, 8, 175), ("64", "small")),          # forward 63 us large, 67 on 128 rows, 57 on 64
    ((768, 512, 64, 100), ("64", "small")),
    ((768, 512, 64, 240), ("128", "small")),
    ((512, 256, 16, 2000), ("large", "small")),       # weight gradients 145 us small, 323 large
]


@pytest.mark.parametrize("shape,want", TIMED)
def test_timed_shapes(shape, want):
    d, I, S, r = shape
    assert plan(d, I, S, 0, r * S // 4, 4) == want


def test_rows_that_must_not_depend_on_the_tile_cover_every_tile():
    for n, tile in G.SAME_ROWS.items():
        c = G.SAME_LAYER
        assert plan(c["d"], c["I"], c["S"], 0, c["S"] * n, 1)[0] == tile
