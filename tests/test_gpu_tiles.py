"""The grouped FFN at the sizes where its tile shapes change: each small tile
(32, 64 and 128 rows), the large one, every pairing with the weight gradients'
tiles, and the int8 forward's, at row, column and k remainders (d and I multiples
of 8, a single token, empty tuning slots, shared experts).  A whole step through
the C ABI against the fp64 oracle on the oracle's routing."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_19078_amd import api, workloads as W
from paper_2508_19078_amd.layer import LayerInputs, MoELayerRunner

import test_gpu_quantized_forward as Q8
from gpu_harness import TOL_FFN, OracleLayer, host, log, rel_fro

pytestmark = pytest.mark.gpu

# fp32: three chained products of at most 1032 terms, each with a rounding error
# of about sqrt(1032) 2^-24 = 2e-6 relative to its norm
TOL_F32 = 1e-5


def _w(T, d, E, k, I, dtype="bf16", ns=0, bias="normal"):
    return W.LayerWorkload(name=f"tiles_{dtype}_{T}_{d}_{E}_{k}_{I}_{ns}", cid=700 + T % 97, T=T, d=d, E=E, k=k, I=I,
                           dtype=dtype, n_shared=ns, bias_kind=bias, bias_var=1.0, zipf_s=1.2)


# r = T (k + shared) / slots and the layer's size decide the row tile and those of
# dW_down and dW_gate/up, named here as fm::tile_plan and fm::dw_tile must choose them
CASES = [
    (_w(1, 72, 4, 2, 40), "32 64 64"),                     # one token, two empty slots, one slab with a remainder
    (_w(33, 200, 6, 2, 136, ns=1), "32 64 64"),            # r = 14
    (_w(130, 264, 8, 4, 136), "64 64 64"),                 # r = 65
    (_w(150, 136, 4, 2, 24, ns=1), "64 64 64"),            # r = 90
    (_w(800, 1032, 64, 8, 264), "64 128 128"),             # r = 100
    (_w(1600, 520, 64, 8, 776, bias="zipf"), "128 128 128"),   # r = 200
    (_w(2400, 520, 64, 8, 776), "large large large"),      # r = 300
    (_w(700, 136, 4, 2, 72), "large 64 64"),               # r = 350
    (_w(1100, 776, 2, 1, 1032), "large 128 128"),          # r = 550, few slots of many tiles
    (_w(5, 1032, 64, 8, 264), "32 128 128"),               # empty slots on 128 x 128 weight-gradient tiles
    (_w(2, 40, 4, 1, 24, "f32"), "32 split split"),        # fp32, empty slots, k below one slab
    (_w(40, 136, 8, 4, 72, "f32", ns=1), "32 split split"),    # r = 22
    (_w(300, 1032, 5, 3, 264, "f32", bias="zipf"), "32 64 64"),   # r = 180, few row tiles
    (_w(700, 136, 4, 2, 72, "f32"), "32 split split"),     # r = 350: ring buffers of the k split reused twice
    (_w(1200, 264, 16, 4, 520, "f32"), "64 64 64"),        # r = 300
    (_w(3, 264, 16, 4, 520, "f32"), "32 64 64"),           # empty slots on 64 x 64 weight-gradient tiles
]


@pytest.mark.parametrize("w", [w for w, _ in CASES], ids=lambda w: w.name)
def test_step(w):
    inp = LayerInputs(w)
    ref = OracleLayer(w, inp)
    r = MoELayerRunner(w, inp)
    r.profile()
    r.merge(counts=torch.from_numpy(ref.counts.astype(np.int32)).cuda())
    log(w.name)
    r.forward(idx=torch.from_numpy(ref.idx.astype(np.int32)).cuda(),
              gate=torch.from_numpy(ref.gate.astype(np.float32)).cuda())
    for t in (r.dWg, r.dWu, r.dWd):
        t.fill_(float("nan"))                    # a gradient is written, not added to what was there
    r.backward(dgate=True)
    u = torch.empty(r.S_r + w.n_shared, dtype=torch.float32, device="cuda")
    api.moe_expert_utility(r.layer_tables, r.x_sq, r.dy_sq, r.perm_token, r.perm_gate, r.offsets, w.T, w.k, r.ws_bwd, u)
    torch.cuda.synchronize()
    tol = TOL_F32 if w.dtype == "f32" else TOL_FFN
    dX, dW, dgate = ref.backward()
    assert rel_fro(host(r.Y), ref.forward()) <= tol
    assert rel_fro(host(r.dX), dX) <= tol
    assert rel_fro(host(r.dgate), dgate) <= tol
    assert rel_fro(host(u), O.expert_utility_rank_one(ref.X, ref.dY, ref.idx, ref.gate, ref.plan.expert_map,
                                                      ref.slots)) <= tol
    once = []
    for i, s in enumerate(r.tuning_slots):
        got = [host(t[i]).copy() for t in (r.dWg, r.dWu, r.dWd)]
        for a, b in zip(got, dW[s]):
            if not np.any(b):
                assert not a.any()               # an empty tuning slot: exact zeros (not NaN)
            else:
                assert rel_fro(a, b) <= tol
        if not np.any(dW[s][0]):
            for t in (r.dWg, r.dWu, r.dWd):      # what an earlier micro-batch left in such a slot stays
                t[i].fill_(3.0)
            got = [np.full_like(a, 1.5) for a in got]
        once.append(got)
    r.backward(accumulate_dw=True)               # the same step again: fp32 x + x
    torch.cuda.synchronize()
    for i, got in enumerate(once):
        for a, t in zip(got, (r.dWg, r.dWu, r.dWd)):
            np.testing.assert_array_equal(host(t[i]), 2 * a)


# (T, d, E, k, I, shared, experts drawn from, sampled rows) of the int8 forward's tiles
Q8_CASES = {
    "tiles_q8_32": (20, 80, 8, 2, 48, 1, 7, None),         # r = 7, an empty slot
    "tiles_q8_64": (260, 144, 6, 2, 112, 0, 6, None),      # r = 87, 12 128-row tiles
    "tiles_q8_128": (1600, 144, 64, 6, 336, 0, 63, None),  # r = 150, 320 128-row tiles; I and d end inside a slab
    "tiles_q8_256": (7100, 4112, 4, 1, 3056, 0, 4, 96),    # r = 1775, the 256-row tile; I and d end inside a slab
}
# rows of each one's row tile
Q8_TILES = {"tiles_q8_32": 32, "tiles_q8_64": 64, "tiles_q8_128": 128, "tiles_q8_256": 256}


@pytest.mark.parametrize("name", list(Q8_CASES))
def test_int8_forward(name, monkeypatch):
    monkeypatch.setitem(Q8.CASES, name, Q8_CASES[name])
    Q8.test_quantised_forward(name)


def _bf16(rng, *shape, std=1.0):
    return torch.from_numpy((std * rng.standard_normal(shape)).astype(np.float32)).to(torch.bfloat16).cuda()


# rows per slot of a call on 32 slots, d = 712, I = 1032: one for each row tile
SAME_ROWS = {5: "32", 40: "64", 200: "128", 300: "large"}
SAME_LAYER = dict(S=32, d=712, I=1032)


def test_rows_do_not_depend_on_the_tile():
    """A row's activations, outputs and gradients are the same bits whichever row
    tile its call takes: a slot's first rows, alone (32-row tiles) and in larger
    calls (64 and 128-row tiles, the large ones), in one ascending-k sum each."""
    S, d, I = (SAME_LAYER[q] for q in "SdI")
    n_min, n_max = min(SAME_ROWS), max(SAME_ROWS)
    rng = np.random.default_rng([77, d, I])
    Wg, Wu, Wd = _bf16(rng, S, I, d, std=d ** -0.5), _bf16(rng, S, I, d, std=d ** -0.5), _bf16(rng, S, d, I, std=I ** -0.5)
    X, dO = _bf16(rng, S, n_max, d), _bf16(rng, S, n_max, d)
    tables = api.LayerTables(d, I, torch.bfloat16, S, 0, *([m[s] for s in range(S)] for m in (Wg, Wu, Wd)),
                             *([None] * S for _ in range(3)), device="cuda")

    def call(n):
        T = S * n
        e = lambda c: torch.full((T, c), float("nan"), dtype=torch.bfloat16, device="cuda")
        u8 = lambda b: torch.empty(b, dtype=torch.uint8, device="cuda")
        off = torch.arange(0, T + 1, n, dtype=torch.int32, device="cuda")
        Xp, dOp = (t[:, :n].reshape(T, d).contiguous() for t in (X, dO))
        out = {"A_g": e(I), "A_u": e(I), "H": e(I), "O": e(d), "dX": e(d)}
        api.moe_grouped_swiglu_fwd(tables, Xp, Xp, off, T, 1, out["A_g"], out["A_u"], out["H"], out["O"],
                                   u8(api.moe_grouped_swiglu_fwd_workspace_size(tables, T, 1)))
        api.moe_grouped_swiglu_bwd(tables, Xp, Xp, off, T, 1, out["A_g"], out["A_u"], out["H"], dOp, out["dX"],
                                   False, u8(api.moe_grouped_swiglu_bwd_workspace_size(tables, T, 1)))
        torch.cuda.synchronize()
        return {q: t.view(S, n, -1)[:, :n_min] for q, t in out.items()}

    want = call(n_max)
    for n in sorted(SAME_ROWS)[:-1]:
        log(f"{n} rows per slot")
        for q, t in call(n).items():
            assert torch.equal(t, want[q]), (n, q)


# layers and rows per slot of the int8 calls compared bit for bit: the row tile of each
Q8_SAME = [(dict(S=16, d=208, I=1040), {5: 32, 70: 64, 300: 128}),
           (dict(S=4, d=4112, I=3056), {100: 64, 600: 128, 1750: 256})]


@pytest.mark.parametrize("layer,rows", Q8_SAME)
def test_int8_rows_do_not_depend_on_the_tile(layer, rows):
    """The same for the int8 forward's row tiles."""
    S, d, I = (layer[q] for q in "SdI")
    n_min, n_max = min(rows), max(rows)
    rng = np.random.default_rng([78, d, I])
    q = [torch.from_numpy(rng.integers(-128, 128, size=sh, dtype=np.int8)).cuda() for sh in ((S, I, d), (S, I, d), (S, d, I))]
    sc = [torch.from_numpy((rng.uniform(0.5, 1.5, size=(S, r)) / (127 * c ** 0.5)).astype(np.float32)).cuda()
          for r, c in ((I, d), (I, d), (d, I))]
    X = _bf16(rng, S, n_max, d)
    tables = api.LayerTablesQ8(d, I, S, 0, *([m[s] for s in range(S)] for m in q + sc), device="cuda")

    def call(n):
        T = S * n
        off = torch.arange(0, T + 1, n, dtype=torch.int32, device="cuda")
        Xp = X[:, :n].reshape(T, d).contiguous()
        H, Ot = (torch.full((T, c), float("nan"), dtype=torch.bfloat16, device="cuda") for c in (I, d))
        ws = torch.empty(api.moe_grouped_swiglu_fwd_q8_workspace_size(tables, T, 1), dtype=torch.uint8, device="cuda")
        api.moe_grouped_swiglu_fwd_q8(tables, Xp, Xp, off, T, 1, H, Ot, ws)
        torch.cuda.synchronize()
        return H.view(S, n, I)[:, :n_min], Ot.view(S, n, d)[:, :n_min]

    want = call(n_max)
    for n in sorted(rows)[:-1]:
        log(f"{n} rows per slot")
        H, Ot = call(n)
        assert torch.equal(H, want[0]) and torch.equal(Ot, want[1]), n
