"""Which tiles the launchers choose for the models of the GPU tests: their comments name a tile and the parts of k for each shape, and a change of a
cost constant must not leave one of them untested without notice.  Host code only."""
import ctypes

import pytest

import paper_2505_11564_amd as hf
import synth_inputs as si
import test_gpu_gemm_f32 as f32
import test_gpu_gemm_f32_split as split
import test_gpu_linear_products as lin

LIN_TILES = ["64x64", "64x128", "128x64", "128x96", "128x128", "128x192", "128x256"]
F32_TILES = ["64x64", "128x128", "32x32"]
WS = 16 << 20  # floats of scratch


def _linear(M, N, K, tb, lo=0, bf16=0, add=0):
    """(tile, parts of k) of a bf16 product with its tangent."""
    r = hf.lib().hf_internal_linear_plan((ctypes.c_int64 * 9)(M, N, K, 0, tb, lo, bf16, add, WS))
    return ("pair", 1) if r < 0 else (LIN_TILES[r % 16], r // 16)


def _f32(*products):
    """Tile and parts of k of fp32 products (M, N, K, terms) launched together."""
    num = (ctypes.c_int64 * (4 * len(products)))(*[x for p in products for x in p])
    parts = (ctypes.c_int * len(products))()
    r = hf.lib().hf_internal_f32_plan(num, len(products), ctypes.c_int64(WS), parts)
    assert r >= 0
    return F32_TILES[r], list(parts)


def _dims(model, batch, seq=None):
    T = batch * (seq or model["max_seq"])
    D, F, V = model["d_model"], model["d_ff"], model["vocab"]
    return T, D, F, V, D // model["n_head"] * model.get("n_kv_head", model["n_head"])


def _linear_plans(model, batch):
    """Every product-rule product of a model in bf16, forward and adjoint."""
    T, D, F, V, Dkv = _dims(model, batch)
    if model["arch"] == "gpt":
        fwd = [(3 * D, D, 1, 0), (D, D, 0, 1), (F, D, 1, 0), (D, F, 0, 1), (V, D, 0, 0)]
        bwd = [(D, V, 0, 0), (F, D, 1, 0), (D, F, 0, 0), (D, D, 1, 0), (D, 3 * D, 0, 0)]
        lo = 0
    else:
        fwd = [(D, D, 0, 0), (Dkv, D, 0, 0), (Dkv, D, 1, 0), (D, D, 0, 1), (F, D, 1, 0), (D, F, 0, 1), (V, D, 0, 0)]
        bwd = [(D, V, 0, 0), (F, D, 1, 0), (D, F, 0, 0), (D, F, 0, 1), (D, D, 1, 0), (D, D, 0, 0), (D, Dkv, 0, 1)]
        lo = 1
    return ({_linear(T, n, k, 0, lo, o, a) for n, k, o, a in fwd}, {_linear(T, n, k, 1, 0, o, a) for n, k, o, a in bwd})


def _f32_plans(model, batch, seq=None):
    """The same in fp32, and the weight gradients, of the linear layers and the head."""
    T, D, F, V, Dkv = _dims(model, batch, seq)
    shapes = [(3 * D, D), (D, D), (F, D), (D, F), (V, D)] if model["arch"] == "gpt" else [(D, D), (Dkv, D), (F, D), (D, F), (V, D)]
    out = set()
    for n, k in shapes:
        for N, K in ((n, k), (k, n)):
            tile, parts = _f32((T, N, K, 1), (T, N, K, 2))
            out.add((tile, "cut" if max(parts) > 1 else "whole"))
    groups = [[(F, D), (D, F)], [(D, D), (D, 3 * D)], [(V, D)]] if model["arch"] == "gpt" else [[(F, D), (D, F), (D, F)], [(D, D)] * 2 + [(D, Dkv)] * 2, [(D, V)]]
    for grp in groups:
        tile, parts = _f32(*[(m, n, T, 2) for m, n in grp])
        out.add((tile, "cut" if max(parts) > 1 else "whole"))
    return out


# what the comments beside the shapes say: (tile, parts of k) of the forward products and of the adjoints
LINEAR = {
    "wide": ({("128x96", 1), ("64x64", 1), ("128x256", 1), ("64x128", 2)}, {("128x256", 1), ("64x128", 2)}),
    "middle": ({("64x128", 1), ("128x128", 1), ("128x64", 4)}, {("128x128", 1), ("128x64", 4)}),
    "long_rows": ({("128x192", 1), ("64x128", 7)}, {("128x192", 1), ("64x128", 7)}),
    "few_rows": ({("64x128", 1), ("64x64", 6)}, {("64x128", 1), ("64x64", 6)}),
    "pairs_long_rows": ({("128x192", 1), ("64x128", 7)}, set()),
    "pairs_middle": ({("128x128", 1), ("64x64", 3)}, {("64x128", 5)}),
    "pairs_few_rows": ({("64x128", 1), ("64x64", 5)}, set()),
    "tiny": ({("64x64", 1)}, {("64x64", 1)}),
    "vocabulary": ({("pair", 1)}, {("128x128", 7)}),
}


@pytest.mark.parametrize("name", list(lin.SHAPES))
def test_linear_products_take_the_tiles_they_are_there_for(name):
    for got, said in zip(_linear_plans(*lin.SHAPES[name]), LINEAR[name]):
        assert said <= got, (said - got, got)


# fp32: tile, k whole or cut, of the models of the two files
F32 = {
    "large": {("128x128", "whole"), ("128x128", "cut"), ("64x64", "cut")},
    "large_unaligned": {("128x128", "whole"), ("128x128", "cut"), ("64x64", "whole"), ("64x64", "cut")},
    "middle": {("64x64", "whole"), ("64x64", "cut")},
    "middle_unaligned": {("64x64", "cut")},
}
F32_MODELS = {
    "cut": {("128x128", "cut"), ("64x64", "cut")},
    "unaligned": {("64x64", "whole"), ("64x64", "cut"), ("32x32", "whole")},
    "large": {("128x128", "whole"), ("64x64", "whole")},
    "whole": {("128x128", "whole")},
    "vocabulary": {("128x128", "whole")},
    "single": {("32x32", "whole")},
    "llama": {("64x64", "cut"), ("32x32", "whole")},
}


@pytest.mark.parametrize("name", list(split.SHAPES))
def test_fp32_products_in_parts_take_the_tiles_they_are_there_for(name):
    got = _f32_plans(*split.SHAPES[name])
    assert F32[name] <= got, (F32[name] - got, got)


@pytest.mark.parametrize("name", list(f32.SHAPES))
def test_fp32_products_take_the_tiles_they_are_there_for(name):
    cfg = f32.SHAPES[name]
    got = _f32_plans(cfg["model"], cfg["batch"], 1 if name == "single" else None)
    assert F32_MODELS[name] <= got, (F32_MODELS[name] - got, got)
