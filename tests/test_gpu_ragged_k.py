"""bf16 products whose k is not a multiple of a slab (64 or 32): token counts and vocabularies with remainders of 1, an odd
number and one short of a slab, through whole Hessian-vector products against the float64 oracle.

Where all widths are multiples of eight, weight gradients contract over rows of zeros up to the next multiple of 64 tokens, and the ragged k left
are those of the vocabulary and of attention; with a d_ff that is none, W_o, W_qkv and the tied head have the number of tokens
itself, alone and (width 264: the rest of a layer goes in launches of its own) as one launch.

Tolerance 2e-2, the bound of bf16 products everywhere (operands rounded to 2^-9), and twice that for every matrix by itself.  In the second
test only the last sequence has labels, its last token too, which is the whole remainder of 65 or 129 (the last position of a text has no label and no
adjoint to be left out): without that token the matrices are 0.07 to 1 off (in float64)."""
import numpy as np
import pytest

import paper_2505_11564_amd as hf
import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

MODEL = dict(gpt=lambda s, v: si._gpt(2, 320, 5, 1288, v, s), llama=lambda s, v: si._llama(1, 256, 4, 696, v, s, n_kv=2))


@pytest.mark.parametrize("arch,batch,seq,vocab", [("gpt", 1, 65, 211), ("gpt", 3, 43, 97), ("gpt", 2, 95, 255), ("llama", 1, 127, 193),
                                                  ("llama", 5, 13, 65)])
def test_hvp_ragged_k(arch, batch, seq, vocab):
    from gpu_util import gpu_hvp, rel_l2
    model = MODEL[arch](seq, vocab)
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=seq)
    v = si.make_direction(len(p), 3)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v, "bf16")
    assert np.isfinite(got).all()
    assert rel_l2(got, want) <= 2e-2


TOKENS = {
    "padded_65": (si._gpt(2, 320, 5, 1288, 97, 5), 13),
    "padded_129": (si._gpt(2, 320, 5, 1288, 97, 3), 43),
    "ragged_65": (si._gpt(2, 320, 5, 1284, 97, 5), 13),
    "ragged_129": (si._gpt(2, 320, 5, 1284, 97, 3), 43),
    "ragged_191": (si._gpt(1, 320, 5, 1284, 97, 1), 191),
    "ragged_llama_65": (si._llama(1, 256, 4, 700, 193, 5, n_kv=2), 13),
    "ragged_group_65": (si._gpt(1, 264, 3, 32508, 97, 5), 13),
    "ragged_group_129": (si._gpt(2, 264, 3, 32508, 97, 3), 43),
    "mlp_65": (si._mlp(64, 128, 10), 65),
    "mlp_129": (si._mlp(72, 200, 40), 129),
    "mlp_191": (si._mlp(264, 264, 264), 191),
}


def _inputs(name):
    model, batch = TOKENS[name]
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    if model["arch"] == "mlp":
        x, y = si.make_batch(dict(model=model, batch=batch, tokens=None))
    else:
        x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=model["max_seq"])
        y[:] = -1
        y[-1] = x[0]  # the last sequence alone, its last token too
    return model, p, x, y, si.make_direction(len(p), 3)


@pytest.mark.parametrize("name", list(TOKENS))
def test_last_token_counts(name):
    from gpu_util import block_errors, gpu_hvp, rel_l2
    model, p, x, y, v = _inputs(name)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    ctx = hf.Context(model, len(x), 0, "bf16")
    for _ in range(2):
        got, _ = gpu_hvp(model, p, x, y, v, "bf16", ctx=ctx)
        assert np.isfinite(got).all()
        assert rel_l2(got, want) <= 2e-2
        for nm, err, _ in block_errors(model, got, want, [e for e in om.layout(model) if len(e[2]) == 2]):
            assert err <= 4e-2, (nm, err)
    ctx.close()
