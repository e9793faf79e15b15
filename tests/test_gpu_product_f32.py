"""Single fp32 products on each tile, where an operand is far from the ordinary: against float64, or against the same product of
ordinary operands where the time is what counts."""
import time

import pytest

pytestmark = pytest.mark.gpu

TILES = [0, 1, 2]  # 64 x 64, 128 x 128 (operands as bf16 parts), 32 x 32


def _randn(*shape, seed=1, scale=1.0):
    import torch
    return torch.randn(*shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda") * scale


def _seconds(fn):
    """The shortest of three calls (the time of a product that ends in a synchronisation)."""
    best = 1e9
    for _ in range(3):
        t = time.perf_counter()
        fn()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("tile", TILES)
def test_padding_that_nobody_wrote(tile, trans):
    """Row-contiguous operands are read up to the next multiple of four columns.  What lies there takes part in no result, and must not
    make a block compute its tile again, which takes many times as long: the product may take five times as long as with zeros there (runs of
    one product differ by far less, a tile computed again one number at a time took a hundred times as long)."""
    import torch
    from gpu_util import fp32_product
    K, N = 30000, 61
    buf = torch.zeros(K, 64, device="cuda")
    buf[:, :N] = _randn(K, N)
    A = _randn(K, 64, seed=2).t() if trans else _randn(64, K, seed=2)
    B = buf[:, :N]
    want = A.double() @ B.double()
    plain = _seconds(lambda: fp32_product(A, B, tile, 1))
    buf[:, N:] = float("nan")
    got = fp32_product(A, B, tile, 1)
    assert (got.double() - want).norm() <= 1e-5 * want.norm()
    assert _seconds(lambda: fp32_product(A, B, tile, 1)) <= 5 * plain


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("tile", TILES)
def test_products_just_below_the_largest_float(tile, sign):
    """Mantissas 1.01967 and 1.96111: their product 1.9997 fits below the largest float, that of the two rounded up to eight bits (2.007)
    does not.  One such product is the whole sum, so the result is it, rounded once."""
    import torch
    from gpu_util import fp32_product
    A, B = torch.zeros(70, 45, device="cuda"), torch.zeros(45, 66, device="cuda")
    A[3:68:13, 40] = sign * 1.01967 * 2.0 ** 63
    B[40, 1:66:9] = 1.96111 * 2.0 ** 64
    want = (A.double() @ B.double()).float()
    assert torch.isfinite(want).all() and want.abs().max() > 3.4e38
    got = fp32_product(A, B, tile, 1)
    assert torch.isfinite(got).all()
    assert ((got - want).abs() <= want.abs() * 2.0 ** -23).all()
