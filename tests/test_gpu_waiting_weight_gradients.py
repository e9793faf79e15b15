"""Weight-gradient products that wait for those of other layers: launches that span layers, the adjoints' buffers taken in turn, the head's
product among them, products cut off by the number a launch holds; through whole products against the float64 oracle.

Tolerance 2e-2, the bound of bf16 products everywhere (operands rounded to 2^-9), and twice that for every matrix by itself; a
product launched after its operands were overwritten, or not at all, is far above it."""
import numpy as np
import pytest

import paper_2505_11564_amd as hf
import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

# model, batch: tiles of 256 x 256 a layer, buffers; what starts the launches (test_waiting_launches_cpu.py holds the comments to it)
SHAPES = {
    "many_products": (si._gpt(6, 264, 3, 1048, 97, 77), 2),             # 32, 4: 16 products fill a launch; six layers go twice round the buffers
    "inside_a_layer": (si._gpt(3, 1000, 10, 4040, 300, 67), 1),         # 192, 3: one launch, of the head and all three layers, at the end
    "odd_head": (si._gpt(5, 512, 8, 2048, 4099, 40, tie=0), 2),         # 48, 4: untied head of odd width; 16 products
    "llama": (si._llama(5, 320, 5, 856, 515, 50), 2),                   # 40, 4: 16 products, two layers and a part
    "llama_grouped": (si._llama(4, 240, 10, 648, 130, 45, n_kv=2), 3),  # stored attention, shared key / value heads; 16 products
    "cut": (si._gpt(7, 128, 2, 512, 97, 301), 4),                       # k in parts, results cleared beforehand; 16 products, without the head
    "three_buffers": (si._gpt(7, 264, 3, 8456, 97, 33), 2),             # 148, 3: each third layer the next one needs the buffers
    "two_buffers": (si._gpt(5, 264, 3, 18440, 97, 33), 2),              # 300, 2: each second layer, for the head's buffer as well
    "full_rounds": (si._gpt(5, 264, 3, 9736, 97, 33), 2),               # 168, 3: a full round after the first, later the second product of a layer
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_products_that_wait(name):
    from gpu_util import block_errors, gpu_hvp, rel_l2
    model, batch = SHAPES[name]
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=model["max_seq"])
    v = si.make_direction(len(p), 5)
    ctx = hf.Context(model, batch, 0, "bf16")
    for rows in (batch, 1):  # the second product finds the first one's adjoints in the buffers
        want = om.hvp(model, p.astype(np.float64), x[:rows], y[:rows], v.astype(np.float64))
        got, _ = gpu_hvp(model, p, x[:rows], y[:rows], v, "bf16", ctx=ctx)
        assert np.isfinite(got).all()
        assert rel_l2(got, want) <= 2e-2
        lay = [e for e in om.layout(model) if len(e[2]) == 2]
        for nm, err, _ in block_errors(model, got, want, lay):
            assert err <= 4e-2, (nm, err)
    ctx.close()
