"""Single bf16 products with their tangents on each tile of the product-rule kernel, k whole and in parts, with and without low-order
halves, ragged in rows, columns and k, against float64.

Tolerance: products of bf16 numbers are exact and their sums round in fp32, sqrt(K / 6) 2^-24 = 1e-6 at K = 1611 (twice that is
allowed); a bf16 result is rounded to 2^-9 at most, its pair to 2^-17."""
import pytest

pytestmark = pytest.mark.gpu

# tile: index in the launcher's table, operand tiles (4, and with one or two low-order halves 5, 6) for which there is a kernel
TILES = {"64x64": (0, (4, 5, 6)), "64x128": (1, (4, 5, 6)), "128x64": (2, (4,)), "128x96": (3, (4,)), "128x128": (4, (4, 5)),
         "128x192": (5, (4, 5)), "128x256": (6, (4,))}
CASES = [(t, n, tr) for t, (_, ns) in TILES.items() for n in ns for tr in ("nn", "nt")] + [(t, 4, "tn") for t in ("64x64", "64x128")]


def _operand(rows, cols, transposed, seed, scale=1.0):
    """bf16, rows padded to 16 bytes with NaN in the padding."""
    import torch
    r, c = (cols, rows) if transposed else (rows, cols)
    buf = torch.full((r, (c + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:, :c] = torch.randn(r, c, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda") * scale
    return buf[:, :c].t() if transposed else buf[:, :c]


@pytest.mark.parametrize("bf16_out", [False, True])
@pytest.mark.parametrize("K,parts", [(1611, 1), (1611, 3), (1600, 3), (128, 1), (9, 1)])
@pytest.mark.parametrize("tile,nt,trans", CASES)
def test_product_and_tangent(tile, nt, trans, K, parts, bf16_out):
    import torch
    from gpu_util import bf16_product
    M, N = 293, 411
    A, At = (_operand(M, K, trans[0] == "t", s) for s in (1, 2))
    B, Bt = (_operand(K, N, trans[1] == "t", s) for s in (3, 4))
    A_lo = _operand(M, K, trans[0] == "t", 5, 2.0 ** -9) if nt >= 5 else None
    B_lo = _operand(K, N, trans[1] == "t", 6, 2.0 ** -9) if nt >= 6 else None
    add, add_t = (None, None) if bf16_out else (torch.randn(M, 416, device="cuda") for _ in range(2))
    got = bf16_product(A, B, At, Bt, A_lo, B_lo, add, add_t, bf16_out, TILES[tile][0], parts)
    d = lambda x: x.double()
    want, want_t = d(A) @ d(B), d(At) @ d(B) + d(A) @ d(Bt)
    if nt >= 5:
        want += d(A_lo) @ d(B)
    if nt >= 6:
        want += d(A) @ d(B_lo)
    if bf16_out:
        C, C_lo, Ct = (d(x) for x in got)
        pairs = [(C, want, 2.0 ** -9), (C + C_lo, want, 2.0 ** -17), (Ct, want_t, 2.0 ** -9)]
    else:
        pairs = [(d(got[0]), want + d(add[:, :N]), 2e-6), (d(got[1]), want_t + d(add_t[:, :N]), 2e-6)]
    for g, w, tol in pairs:
        assert (g - w).norm() <= tol * w.norm()


@pytest.mark.parametrize("M,N", [(512, 16384), (500, 16300), (1900, 3960), (512, 28672)])
def test_low_order_halves_in_even_rounds_of_large_tiles(M, N):
    """One and two rounds of 256 x 256 tiles: the product with its low-order half and the tangent as two products of one launch."""
    import torch
    from gpu_util import bf16_product
    from test_product_plans_cpu import _linear
    K = 520
    assert _linear(M, N, K, 0, lo=1) == ("pair", 1)
    A, At, A_lo = (_operand(M, K, False, s, c) for s, c in ((1, 1.0), (2, 1.0), (3, 2.0 ** -9)))
    B, Bt = (_operand(K, N, False, s) for s in (4, 5))
    got = bf16_product(A, B, At, Bt, A_lo)
    d = lambda x: x.double()
    for g, w in zip(got, ((d(A) + d(A_lo)) @ d(B), d(At) @ d(B) + d(A) @ d(Bt))):
        assert (d(g) - w).norm() <= 2e-6 * w.norm()
