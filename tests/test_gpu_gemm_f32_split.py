"""fp32 products whose operands are taken apart into three bf16 numbers: the edges of their two tiles, aligned and not, against
the float64 oracle; sums of many products; numbers that round to infinity in bf16.

Tolerance: the parts carry all 24 bits of an operand and the terms left out are at most 2^-24 of a product (both mantissas just above 1;
2^-27.5 on average), so what remains is the rounding of the sums: runs of at most 1024 k in 16-term instructions, added up over the
runs: sqrt(64 / 6) 2^-24 of a run and sqrt(runs / 6) 2^-24 of their sum, below 3e-7 for a product of 50000; a dozen products between input
and result, the elementwise passes between them as well, add up in quadrature to less than 2e-6."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

SHAPES = {
    # 128 x 128 tiles, ragged in rows and columns and with a ragged k; a head of many slabs, in parts
    "large": (si._gpt(1, 516, 4, 2068, 20011, 263), 4),
    # the same, no row 16-byte aligned
    "large_unaligned": (si._gpt(1, 517, 11, 2071, 1003, 261), 4),
    # 64 x 64 tiles whole and in parts
    "middle": (si._gpt(2, 324, 3, 1300, 515, 131), 3),
    # in parts, no row aligned
    "middle_unaligned": (si._llama(1, 330, 3, 1309, 513, 131, n_kv=1), 3),
}


def _inputs(name):
    model, batch = SHAPES[name]
    p = si.make_params(model, perturb=0.1)
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=model["max_seq"])
    return model, p, x, y


@pytest.mark.parametrize("name", list(SHAPES))
def test_hvp_against_64_bits(name):
    from gpu_util import gpu_hvp, rel_l2
    model, p, x, y = _inputs(name)
    v = si.make_direction(len(p), 4)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v)
    assert rel_l2(got, want) <= 2e-6


@pytest.mark.parametrize("name", ["large", "middle_unaligned"])
def test_a_number_that_rounds_to_infinity(name):
    """3.4e38 is finite in fp32 and infinite in bf16.  The product is linear in the direction, so the column of one weight scaled by
    it is the answer; the gain in front of that weight is small, so that nothing overflows fp32 on the way."""
    from gpu_util import gpu_hvp, rel_l2
    model, p, x, y = _inputs(name)
    lay = {nm: (off, sh) for nm, off, sh in om.layout(model)}
    big = np.float32(3.4e38)
    gpt = model["arch"] == "gpt"
    off, sh = lay["h0.Wfc" if gpt else "h0.Wup"]
    j = off + 5 * sh[1] + 7
    p[lay["h0.ln2.g" if gpt else "h0.rms2.g"][0] + 5] = 1e-6
    if gpt:
        p[lay["h0.ln2.b"][0] + 5] = 0.0
    v = np.zeros(len(p), np.float32)
    v[j] = 1.0
    column, _ = gpu_hvp(model, p, x, y, v)
    v[j] = big
    got, _ = gpu_hvp(model, p, x, y, v)
    assert np.isfinite(got).all()
    assert rel_l2(got / float(big), column) <= 2e-6
