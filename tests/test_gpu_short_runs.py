"""Runs with an MLP whose iterations are enqueued ahead: the update that adds the product's shares itself (few of them), and the separate sum
(many); products of one and of two waves a sample.  Runs agree with single steps bit for bit (nothing in either depends on timing), products
with the float64 oracle to 1e-5 (fp32 sums of at most a few thousand terms, as in test_gpu_small_runs.py)."""
import numpy as np
import pytest
import torch

import paper_2505_11564_amd as hf
import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu


def _inputs(sizes, batch):
    model = si._mlp(*sizes)
    p = si.make_params(model)
    x, y = si.make_batch(dict(model=model, batch=batch, tokens=None))
    return model, p, x, y


# 32-32-10: 1386 parameters, so 47 blocks of eight samples are the most that the update adds
@pytest.mark.parametrize("sizes,batch,reorth,m", [((32, 32, 10), 376, "full", 9), ((32, 32, 10), 377, "full", 9), ((32, 32, 10), 377, "none", 9),
                                                  ((1, 1, 2), 1, "full", 2), ((64, 64, 10), 100, "full", 20), ((64, 64, 10), 256, "none", 6)])
def test_runs_equal_single_steps(sizes, batch, reorth, m):
    model, p, x, y = _inputs(sizes, batch)
    pd, xd, yd = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p, x, y))
    zd = torch.from_numpy(si.make_probe(len(p), 0)).cuda()
    ctx = hf.Context(model, batch, m, "f32", "f32" if reorth == "full" else "none")
    res = ctx.hf_slq(pd, xd, yd, batch, 1, zd, 1, m, reorth)
    q_run, q_step = torch.empty(ctx.n, device="cuda"), torch.empty(ctx.n, device="cuda")
    ctx.hf_lanczos_get_vector(0, q_run)
    ctx.hf_lanczos_init(zd, reorth)
    steps = [ctx.hf_lanczos_step(pd, xd, yd, batch, 1) for _ in range(m)]
    ctx.hf_lanczos_get_vector(0, q_step)
    np.testing.assert_array_equal(res["alpha"][0], [s[0] for s in steps])
    np.testing.assert_array_equal(res["beta"][0], [s[1] for s in steps])
    assert torch.equal(q_run, q_step)
    ctx.close()


# hidden units and classes on both sides of 8, 16, 32 and 64 lanes; from 2049 samples one wave a sample, unless LDS holds no sixteen
@pytest.mark.parametrize("sizes,batch", [((8, 8, 8), 2049), ((9, 9, 16), 2048), ((31, 17, 17), 2050), ((5, 33, 32), 4097), ((70, 64, 33), 2049),
                                         ((40, 65, 65), 3000), ((200, 30, 100), 2060), ((256, 48, 2), 2049)])
def test_products(sizes, batch):
    from gpu_util import gpu_hvp, rel_l2
    model, p, x, y = _inputs(sizes, batch)
    y[5:9] = -1
    v = si.make_direction(len(p), 2)
    want_loss, _, want, _ = om.loss_grad_hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, loss = gpu_hvp(model, p, x, y, v)
    assert rel_l2(got, want) <= 1e-5
    assert abs(loss - want_loss) <= 1e-5 * abs(want_loss)
