"""bf16 product-rule products (a product and its tangent in one launch) at each tile the launcher chooses from, with k whole and
in parts, ragged in rows, columns and k, through whole Hessian-vector products against the float64 oracle.  (test_product_plans_cpu.py
holds the launcher to the tiles named here.)

Tolerance 2e-2, the bound of bf16 products everywhere (operands rounded to 2^-9), also for every parameter tensor's block on its
own where it carries more than 1e-6 of the whole: a wrong tile of one product is a tenth of some block."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

# model, batch: tiles (and parts of k) of its layers' products
SHAPES = {
    # 128 x 96, 64 x 64, 128 x 256, 64 x 128 in two parts
    "wide": (si._gpt(1, 1024, 16, 8200, 97, 385), 2),
    # 64 x 128, 128 x 128, 128 x 64 in four parts
    "middle": (si._gpt(1, 392, 7, 3080, 515, 515), 2),
    # 128 x 192, 64 x 128 in seven parts
    "long_rows": (si._gpt(1, 200, 5, 5176, 97, 275), 4),
    # 64 x 128, 64 x 64 in six parts
    "few_rows": (si._gpt(1, 200, 5, 3576, 97, 130), 4),
    # with low-order halves: 128 x 192, 64 x 128 in seven parts
    "pairs_long_rows": (si._llama(1, 208, 2, 5176, 97, 275, n_kv=1), 4),
    # 128 x 128, 64 x 64 in three parts; adjoint: 64 x 128 in five parts
    "pairs_middle": (si._llama(1, 520, 5, 6200, 515, 103, n_kv=5), 5),
    # 64 x 128, 64 x 64 in five parts
    "pairs_few_rows": (si._llama(1, 264, 3, 3576, 97, 103, n_kv=1), 5),
    # fewer rows and columns than a tile, k shorter than a slab and just beyond one
    "tiny": (si._gpt(1, 40, 1, 72, 33, 9), 1),
    # head: more than 1024 blocks of 256 x 256 (primal product and tangent as two products of one launch), and its adjoint:
    # 128 x 128 in seven parts
    "vocabulary": (si._gpt(1, 512, 8, 520, 35003, 260), 4),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_hvp_linear_products(name):
    from gpu_util import block_errors, gpu_hvp, rel_l2
    model, batch = SHAPES[name]
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=model["max_seq"])
    v = si.make_direction(len(p), 7)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v, "bf16")
    assert np.isfinite(got).all()
    assert rel_l2(got, want) <= 2e-2
    total = float(np.linalg.norm(want))
    bad = [r for r in block_errors(model, got, want, om.layout(model)) if r[2] > 1e-6 * total and not r[1] <= 2e-2]
    assert not bad, bad
