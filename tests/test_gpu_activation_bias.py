"""The bias block of H v that the activation's backward pass sums: edges of its 256 columns and of its rows per block, and
the widths that take two launches, against the float64 oracle.

Tolerance of the block on its own: 1e-5 in fp32 and 2e-2 in bf16, the bounds of whole products; a row or a column left out or
taken twice is at least 1 / sqrt(rows or columns) of it, above 4e-3 (fp32) and, at the sizes given to bf16, above 5e-2."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

# width, heads, ffn, sequence, batch
SHAPES = {
    "two_rows": ((8, 1, 264, 2), 1, ("f32", "bf16")),          # fewer rows than a block takes at a time
    "columns_257": ((8, 1, 264, 13), 3, ("f32", "bf16")),      # 8 columns in the second block, a ragged last row group
    "not_by_8": ((12, 1, 260, 13), 3, ("f32", "bf16")),        # two launches
    "16_rows": ((16, 2, 2056, 229), 4, ("f32",)),              # 16 rows a block, the last block ragged
    "32_rows": ((16, 2, 2056, 241), 16, ("f32",)),             # 32 rows a block, the last block ragged
}


@pytest.mark.parametrize("name,dtype", [(n, d) for n in SHAPES for d in SHAPES[n][2]])
def test_bias_block(name, dtype):
    from gpu_util import gpu_hvp, rel_l2
    (width, heads, ffn, seq), batch, _ = SHAPES[name]
    model = si._gpt(1, width, heads, ffn, 33, seq)
    p = si.make_params(model, param_dtype=dtype, perturb=0.1)
    if dtype == "bf16":
        p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(p))
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=seq)
    v = si.make_direction(len(p), 3)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v, dtype)
    tol = 1e-5 if dtype == "f32" else 2e-2
    assert np.isfinite(got).all()
    assert rel_l2(got, want) <= tol
    off, sh = {nm: (o, s) for nm, o, s in om.layout(model)}["h0.bfc"]
    assert rel_l2(got[off:off + sh[0]], want[off:off + sh[0]]) <= tol
