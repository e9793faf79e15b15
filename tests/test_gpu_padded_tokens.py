"""bf16 products over numbers of tokens that are and are not multiples of 64, in turn on one context: the rows behind the tokens, over which the
weight gradients contract too, hold other products' values until they are cleared.  Against the float64 oracle; tolerance 2e-2, as all bf16
products, and twice that for every matrix by itself."""
import numpy as np
import pytest

import paper_2505_11564_amd as hf
import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

MODELS = {
    "gpt": si._gpt(2, 72, 3, 200, 97, 64),
    "llama": si._llama(2, 96, 3, 256, 131, 64),                # streamed attention
    "llama_grouped": si._llama(1, 80, 10, 216, 130, 64, n_kv=2),  # stored attention
    "odd_width": si._gpt(1, 36, 2, 60, 11, 64),                # not a multiple of eight: no padding
}


@pytest.mark.parametrize("name", list(MODELS))
def test_changing_numbers_of_tokens(name):
    import torch
    from gpu_util import block_errors, gpu_hvp, rel_l2
    model = MODELS[name]
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    v = si.make_direction(len(p), 5)
    ctx = hf.Context(model, 3, 0, "bf16")
    want = {}
    for batch, seq in ((3, 64), (3, 21), (2, 64), (3, 21), (1, 1), (1, 64), (3, 63), (3, 21)):
        x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=seq)
        if seq == 1:
            y[:] = 3
        if (batch, seq) not in want:
            want[batch, seq] = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
        got, _ = gpu_hvp(model, p, x, y, v, "bf16", ctx=ctx)
        assert np.isfinite(got).all()
        assert rel_l2(got, want[batch, seq]) <= 2e-2
        for nm, err, den in block_errors(model, got, want[batch, seq], [e for e in om.layout(model) if len(e[2]) == 2]):
            assert err <= 4e-2 or den < 1e-3 * np.linalg.norm(want[batch, seq]), (batch, seq, nm, err)
    ctx.close()
