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


def _special(K, trans):
    """Operands with an infinity, a NaN and a number that rounds to infinity in bf16, each in a row (A) or a column (B) of its own."""
    A, B = _randn(150, K, seed=3), _randn(K, 145, seed=4)
    A[5, K // 3], A[77, 1], A[140, K - 1] = float("inf"), float("nan"), 3.4e38
    B[K - 2, 9], B[0, 130] = -float("inf"), float("nan")
    B[K - 1] *= 1e-3
    return (A.t().contiguous().t(), B.t().contiguous().t()) if trans else (A, B)


@pytest.mark.parametrize("parts", [1, 3])
@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("K", [397, 30000])
@pytest.mark.parametrize("tile", TILES)
def test_operands_that_are_not_finite(tile, K, trans, parts):
    """Infinities and NaN where float64 has them (with a finite operand's 3.4e38 below the overflow), everything else within the rounding of
    a sum one product at a time, sqrt(K / 6) 2^-24 of its size (4.2e-6 for the longest; twice that is allowed), and in at most ten times the time of
    ordinary operands (fp32 instructions after the others: three to four times; one number at a time it was 200 times)."""
    import torch
    from gpu_util import fp32_product
    plain = (_randn(150, K, seed=3), _randn(K, 145, seed=4))
    if trans:
        plain = tuple(x.t().contiguous().t() for x in plain)
    A, B = _special(K, trans)
    want = A.double() @ B.double()
    got = fp32_product(A, B, tile, parts)
    fin = torch.isfinite(want)
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[~fin & ~torch.isnan(want)].double(), want[~fin & ~torch.isnan(want)])
    rows = torch.ones(150, dtype=torch.bool, device="cuda")
    rows[140] = False  # 3.4e38 times a number of its own column: the rest of that row's sums is below the last bit
    for r in (rows, ~rows):
        e, w = (got.double() - want)[r][fin[r]], want[r][fin[r]]
        assert e.norm() <= 8.4e-6 * w.norm()
    if K > 1000:
        assert _seconds(lambda: fp32_product(A, B, tile, parts)) <= 10 * _seconds(lambda: fp32_product(*plain, tile, parts))


@pytest.mark.parametrize("scale", [1e-20, 1e-35, 1e-37, 1e-40, 1e12, 1e24])
@pytest.mark.parametrize("tile", TILES)
def test_operands_of_any_size(tile, scale):
    """Both operands in turn: every float keeps all of its bits, so the error is that of the sum, sqrt(300 / 6) 2^-24 = 4.2e-7 (twice that is
    allowed) whatever the scale.  The other operand is of a size that keeps the result among the normal numbers (with 1e12 and 1e24: sums on
    both sides of 1.2e24, where a tile of parts is computed again)."""
    import torch
    from gpu_util import fp32_product
    A, B = _randn(131, 300, seed=5, scale=scale), _randn(300, 133, seed=6, scale=1e6 if scale < 1 else 1e12)
    for a, b in ((A, B), (B.t(), A.t()), (B.t().contiguous(), A.t().contiguous())):
        want = a.double() @ b.double()
        got = fp32_product(a, b, tile, 1)
        assert (got.double() - want).norm() <= 8.4e-7 * want.norm()


def _mantissas_that_lose_most():
    """A number near 1 whose square loses most when the products of a second with a third part are left out: about 2^-24 of it."""
    import torch
    x = (1 + 0.02 * torch.rand(1 << 20, dtype=torch.float64, generator=torch.Generator().manual_seed(7))).float()
    x0 = x.bfloat16().float()
    x1 = (x - x0).bfloat16().float()
    lost = (2 * x1 * (x - x0 - x1)).double() / x.double() ** 2
    assert 0.9 * 2.0 ** -24 < lost.max() < 1.1 * 2.0 ** -24
    return float(x[lost.argmax()])


@pytest.mark.parametrize("kind", ["normal", "near one", "near one, signs", "most lost", "most lost, signs"])
@pytest.mark.parametrize("K", [16, 64, 128, 512, 1024, 4096])
@pytest.mark.parametrize("tile", [0, 1])
def test_parts_add_up_to_no_more_error_than_the_sum(tile, K, kind):
    """The large products are added 16 at a time, in runs of 1024 k: sqrt(min(K, 1024) / 16 / 6) 2^-24 of rounding in a run (each
    addition rounds a partial sum that grows like a random walk), sqrt(K / 1024 / 6) 2^-24 where the runs are added, 0.7 2^-24 for the last
    rounding and the small products, and up to 2^-24 for those left out where every mantissa loses most (2^-27.5 on average)."""
    import numpy as np
    import torch
    from gpu_util import fp32_product
    g = torch.Generator(device="cuda").manual_seed(K)
    sign = lambda *s: (torch.randint(0, 2, s, generator=g, device="cuda") * 2 - 1).float()
    def draw(*s):
        if kind == "normal":
            return torch.randn(*s, generator=g, device="cuda")
        x = 1 + 0.02 * torch.rand(*s, generator=g, device="cuda") if "near" in kind else torch.full(s, _mantissas_that_lose_most(), device="cuda")
        return x * sign(*s) if "signs" in kind else x
    A, B = draw(192, K), draw(K, 192)
    want = A.double() @ B.double()
    got = fp32_product(A, B, tile, 1)
    bound = np.sqrt(min(K, 1024) / 96 + K / 6144) + 0.7 + (1.0 if "lost" in kind else 0.0)
    assert (got.double() - want).norm() <= bound * 2.0 ** -24 * want.norm()
