"""fp32 products on the matrix cores, through whole Hessian-vector products against the float64 oracle, at the sizes
where their tiles, the parts of a cut k and the unaligned loads can go wrong.

Tolerance: a sum of K terms in fp32, one after the other, carries about sqrt(K / 6) 2^-24 of relative error (each addition
rounds a partial sum that grows like a random walk): 3e-6 at K = 16000 and 5e-6 at the longest here, the adjoint of a head of
40003 columns; the dozen products between input and result with K below 11000 (2.5e-6) add up in quadrature to 9e-6, so 1e-5
holds with room (measured: below 1e-6)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import models as om

pytestmark = pytest.mark.gpu

SHAPES = {
    # ragged last rows and columns: k is cut into parts on both larger tiles, also with a ragged last slab
    "cut": dict(model=si._gpt(1, 520, 4, 2084, 101, 500), batch=2, tokens="zipf"),
    # no row of any operand is 16-byte aligned
    "unaligned": dict(model=si._gpt(1, 261, 9, 1031, 103, 333), batch=3, tokens="zipf"),
    # thousands of 64 x 64 tiles, and 128 x 128 tiles with k whole, ragged in both directions
    "large": dict(model=si._gpt(1, 260, 4, 4100, 97, 515), batch=4, tokens="zipf"),
    # so many tiles that the 128 x 128 one is taken with k whole, ragged in both directions: neither and B transposed,
    "whole": dict(model=si._gpt(1, 132, 3, 10260, 97, 515), batch=4, tokens="zipf"),
    # and a transposed A
    "vocabulary": dict(model=si._gpt(1, 132, 3, 388, 40003, 515), batch=2, tokens="zipf"),
    # one token, one tile, k shorter than a slab
    "single": dict(model=si._llama(1, 8, 2, 20, 17, 4), batch=1, tokens="zipf"),
    # grouped key / value heads: four weight gradients of different widths in a launch
    "llama": dict(model=si._llama(2, 384, 6, 1028, 205, 200, n_kv=2), batch=2, tokens="zipf"),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_hvp_fp32_products(name):
    from gpu_util import gpu_hvp, rel_l2
    cfg = SHAPES[name]
    model = cfg["model"]
    seq = 1 if name == "single" else model["max_seq"]
    p = si.make_params(model, perturb=0.1)
    x, y = si.make_batch(cfg, seq=seq)
    y[0, 0] = 3  # (a single token has no successor to predict)
    v = si.make_direction(len(p), 4)
    want = om.hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, _ = gpu_hvp(model, p, x, y, v)
    assert rel_l2(got, want) <= 1e-5


def test_accumulate_fp32_adds_cut_products_to_the_result():
    import torch
    import paper_2505_11564_amd as hf
    from gpu_util import rel_l2
    from oracle import dataset_hvp
    model = SHAPES["cut"]["model"]
    p = si.make_params(model)
    x, y = si.make_batch(SHAPES["cut"], batch=3, seq=500)
    v = si.make_direction(len(p), 6)
    ctx = hf.Context(model, 2, 0, "f32")
    dev = [torch.from_numpy(a).cuda() for a in (p, x, y, v)]
    out = torch.full((ctx.n,), float("nan"), device="cuda")
    ctx.hf_hvp_accumulate(dev[0], dev[1], dev[2], 3, 2, 500, dev[3], out)
    want, _ = dataset_hvp.hvp_dataset(model, p.astype(np.float64), dataset_hvp.split_batches(x, y, 2), v.astype(np.float64))
    assert rel_l2(out.cpu().numpy().astype(np.float64), want) <= 1e-5
    ctx.close()


def test_spectrum_run_with_cancelling_coefficients():
    """alpha_k = <q_k, H q_k> can cancel to a small part of ||H q_k||, of which a product may be 1e-5 off: 1e-3 of alpha where two
    correct evaluations differ by 1e-6 of the product.  So everything is measured in the operator's scale.  Later vectors
    are off by the earlier coefficients' errors, and a Ritz value by at most the sum of three entries' of T: a few times that."""
    import torch
    import paper_2505_11564_amd as hf
    from oracle import lanczos as olz
    model = si._llama(8, 128, 2, 336, 15251, 40)
    p = si.make_params(model)
    x, y = si.make_batch(dict(model=model, batch=2, tokens="zipf"), seq=40)
    z = si.make_probe(len(p), 2)
    ctx = hf.Context(model, 2, 4, "f32")
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p, x, y, z)]
    r = ctx.hf_slq(dev[0], dev[1], dev[2], 2, 40, dev[3], 1, 4, "none")
    ctx.close()
    alpha, beta, _ = olz.lanczos(lambda q: om.hvp(model, p.astype(np.float64), x, y, q), z.astype(np.float64), 4, "none")
    scale = np.sqrt(alpha ** 2 + beta ** 2 + np.append(0.0, beta[:-1]) ** 2).max()
    assert abs(alpha[0]) < 1e-3 * beta[0] and np.abs(alpha).max() < 0.1 * scale  # what the test is about
    for got, want in ((r["alpha"][0], alpha), (r["beta"][0], beta), (r["ritz"][0], olz.slq_readout(alpha, beta)[0])):
        np.testing.assert_allclose(got, want, rtol=0, atol=4e-5 * scale)
