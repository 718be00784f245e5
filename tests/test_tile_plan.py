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


def dw_tiles(d, I, S, ns, T, k, dtype="bf16"):
    """The small tiles of dW_down and dW_gate/up."""
    f = getattr(api.lib(), "_ZN2fm7dw_tileEPK9moe_layeriib")     # fm::dw_tile(const moe_layer*, int, int, bool)
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    L = api.moe_layer(d, I, api.MOE_BF16 if dtype == "bf16" else api.MOE_F32, S, ns, *[None] * 6)
    return tuple(("split", "64", "128")[f(ctypes.addressof(L), T, k, gate_up)] for gate_up in (False, True))


def q8_rows(d, I, S, ns, T, k):
    """Rows of the int8 forward's row tile."""
    f = getattr(api.lib(), "_ZN2fm7q8_tileEPK12moe_layer_q8ii")   # fm::q8_tile(const moe_layer_q8*, int, int)
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    L = api.moe_layer_q8(d, I, S, ns, *[None] * 6)
    return f(ctypes.addressof(L), T, k)


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
    ((2048, 1408, 8, 4000), ("large", "large")),      # backward 1170 us large, 1387 small
    ((2048, 688, 12, 4000), ("large", "large")),      # 1065, 1180
    ((2048, 1408, 4, 4000), ("large", "small")),      # 796, 740
    ((768, 512, 32, 4000), ("large", "small")),       # 1280, 1135
    ((712, 280, 98, 2315), ("large", "small")),       # Zipf 1981, 1734
]


@pytest.mark.parametrize("shape,want", TIMED)
def test_timed_shapes(shape, want):
    d, I, S, r = shape
    k = 4 if S > 4 else 1
    assert plan(d, I, S, 0, r * S // k, k) == want


# The same of layers whose every slot holds every token: weight gradients
FULL_TIMED = [
    ((984, 2376, 3, 20000), "large"),      # backward 2026 us large, 2377 small
    ((2048, 1408, 2, 1500), "small"),      # r = 2000: 202, 195
    ((2048, 1408, 2, 8000), "large"),      # 598, 676
    ((768, 2048, 3, 4000), "large"),       # 354, 374
    ((1024, 1024, 3, 20000), "small"),     # 1231, 1087
]


@pytest.mark.parametrize("shape,want", FULL_TIMED)
def test_timed_full_slots(shape, want):
    d, I, S, T = shape
    assert plan(d, I, S, 0, T, S)[1] == want
    assert plan(d, I, 0, S, T, 1)[1] == want            # shared experts only


# Rows per slot and the small tiles of dW_down and dW_gate/up
DW_TIMED = [
    ((984, 2376, 3, 400), ("64", "64")),
    ((984, 2376, 3, 16000), ("128", "128")),          # backward 2130 us, 3130 on 64 x 128 tiles
    ((4096, 256, 8, 2000), ("128", "128")),           # 365, 419
    ((1024, 512, 16, 8000), ("64", "128")),
    ((256, 256, 64, 2000), ("64", "64")),             # 520, 474 (Zipf 857, 692)
    ((2048, 1408, 64, 96), ("128", "128")),
]


@pytest.mark.parametrize("shape,want", DW_TIMED)
def test_timed_weight_gradient_shapes(shape, want):
    d, I, S, r = shape
    assert dw_tiles(d, I, S, 0, r * S, 1) == want


# The int8 forward, gate-up + down in us on 128 and 256 rows
Q8_TIMED = [
    ((2048, 1408, 64, 512), 128),     # 615, 645
    ((2048, 1408, 64, 2048), 256),    # 2314, 2214
    ((2048, 1408, 64, 4096), 256),    # 4665, 4278
    ((4096, 1024, 64, 4096), 256),    # 6945, 6203
    ((4096, 2816, 8, 512), 128),      # 290, 305
    ((4096, 2816, 8, 2048), 256),     # 1034, 996
    ((4096, 688, 16, 2048), 128),     # 638, 690
    ((1024, 512, 32, 8192), 128),     # 936, 981
    ((4096, 2816, 4, 2000), 256),     # 569, 552
    ((1024, 1024, 16, 5000), 128),    # 566, 596
    ((1024, 1024, 16, 10000), 256),   # 1114, 1072
    ((976, 2368, 3, 20000), 128),     # 952, 954
]


@pytest.mark.parametrize("shape,want", Q8_TIMED)
def test_timed_int8_shapes(shape, want):
    d, I, S, r = shape
    assert q8_rows(d, I, S, 0, r * S // 8, 8) == want


def test_rows_that_must_not_depend_on_the_tile_cover_every_tile():
    for n, tile in G.SAME_ROWS.items():
        c = G.SAME_LAYER
        assert plan(c["d"], c["I"], c["S"], 0, c["S"] * n, 1)[0] == tile
    for c, rows in G.Q8_SAME:
        for n, tile in rows.items():
            assert q8_rows(c["d"], c["I"], c["S"], 0, c["S"] * n, 1) == tile


@pytest.mark.parametrize("w,want", G.CASES, ids=lambda x: getattr(x, "name", None))
def test_step_cases_take_their_tiles(w, want):
    rows, dw = plan(w.d, w.I, w.E, w.n_shared, w.T, w.k, w.dtype)
    got = (rows,) + (("large",) * 2 if dw == "large" else dw_tiles(w.d, w.I, w.E, w.n_shared, w.T, w.k, w.dtype))
    assert " ".join(got) == want


@pytest.mark.parametrize("name", list(G.Q8_TILES))
def test_int8_cases_take_their_tile(name):
    T, d, E, k, I, ns, _, _ = G.Q8_CASES[name]
    assert q8_rows(d, I, E, ns, T, k) == G.Q8_TILES[name]
