"""The weight-gradient products of one or two layers in one launch, in each of its plans (128 x 128 and 256 x 256 tiles, k whole or cut
into parts; test_waiting_launches_cpu.py holds the models to them), writing and adding, through whole products against the float64 oracle.
A ragged k, which these widths do not have, is in test_gpu_ragged_k.py.

Tolerance 2e-2, the bound of bf16 products everywhere (operands rounded to 2^-9); a wrong or missing tile of a weight
gradient is far above it."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

# model, batch: tiles and parts of k that the estimate chooses; the products contract over the next multiple of 64 tokens
SHAPES = {
    "128_whole": (si._gpt(1, 264, 3, 1048, 97, 77), 2),        # ragged tiles, 154 tokens: fewer slabs than a part needs
    "128_cut": (si._gpt(2, 192, 3, 776, 97, 301), 4),          # two layers, parts of 1204 tokens; ragged tiles
    "256_whole": (si._gpt(1, 1000, 10, 4040, 97, 67), 2),      # more than one round of 128 x 128 tiles
    "256_cut": (si._gpt(1, 512, 8, 3336, 97, 344), 16),        # long k, between 65 and 128 tiles of 256 x 256
}


def _inputs(name):
    model, batch = SHAPES[name]
    p = si.bf16_bits_to_f32(si.f32_to_bf16_bits(si.make_params(model, param_dtype="bf16", perturb=0.1)))
    x, y = si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=model["max_seq"])
    return model, batch, p, x, y, si.make_direction(len(p), 5)


@pytest.mark.parametrize("name", list(SHAPES))
def test_hvp_plans(name):
    from gpu_util import gpu_hvp, rel_l2
    model, batch, p, x, y, v = _inputs(name)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v, "bf16")
    assert np.isfinite(got).all()
    assert rel_l2(got, want) <= 2e-2


@pytest.mark.parametrize("name", ["128_whole", "128_cut", "256_whole"])
def test_accumulate_adds(name):
    import torch
    import paper_2505_11564_amd as hf
    from gpu_util import rel_l2
    from oracle import dataset_hvp
    model, batch, p, x, y, v = _inputs(name)
    ctx = hf.Context(model, batch - 1, 0, "bf16")  # a micro-batch and one sample more
    pd = torch.from_numpy(p).cuda().to(torch.bfloat16)
    xd, yd, vd = (torch.from_numpy(a).cuda() for a in (x, y, v))
    out = torch.full((ctx.n,), float("nan"), device="cuda")
    ctx.hf_hvp_accumulate(pd, xd, yd, batch, batch - 1, model["max_seq"], vd, out)
    want, _ = dataset_hvp.hvp_dataset(model, p.astype(np.float64), dataset_hvp.split_batches(x, y, batch - 1), v.astype(np.float64))
    assert rel_l2(out.cpu().numpy().astype(np.float64), want) <= 2e-2
    ctx.close()
