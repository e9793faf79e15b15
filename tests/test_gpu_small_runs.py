"""The one-kernel MLP product and the one-block Lanczos update at the edges of what they take: more outputs or
hidden units than lanes, samples that fill no block, more samples than blocks, sizes just inside and outside the
limits, and runs that the host enqueues ahead of their results.

Tolerances: products as in test_gpu_gemm_f32.py (fp32 sums of at most a few thousand terms, 1e-5); early Lanczos
coefficients 1e-5 of the iteration's scale (fp32 vectors, fp64 sums)."""
import numpy as np
import pytest
import torch

import paper_2505_11564_amd as hf
import synth_inputs as si
from oracle import lanczos as olz
from oracle import models as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,batch", [((1, 1, 2), 1), ((13, 33, 65), 37), ((100, 70, 31), 1000), ((256, 30, 64), 520),
                                         ((256, 256, 100), 64), ((7, 5, 3), 20000), ((128, 64, 10), 2055), ((7, 5, 3), 65536),
                                         ((7, 5, 3), 65537)])
def test_mlp_product(sizes, batch):
    from gpu_util import gpu_hvp, rel_l2
    model = si._mlp(*sizes)
    cfg = dict(model=model, batch=batch, tokens=None)
    p = si.make_params(model)
    x, y = si.make_batch(cfg)
    if batch > 8:
        y[3:6] = -1
    v = si.make_direction(len(p), 2)
    want_loss, _, want, _ = om.loss_grad_hvp(model, p.astype(np.float64), x, y, v.astype(np.float64))
    got, loss = gpu_hvp(model, p, x, y, v)
    assert rel_l2(got, want) <= 1e-5
    assert abs(loss - want_loss) <= 1e-5 * abs(want_loss)


def _case():
    cfg = si.CONFIGS["mlp_tiny"]
    p = si.make_params(cfg["model"])
    x, y = si.make_batch(cfg)
    return cfg["model"], p, x, y, [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p, x, y)]


@pytest.mark.parametrize("reorth,basis,m", [("full", "f32", 1), ("full", "f32", 2), ("full", "f32", 12), ("none", "none", 9),
                                            ("none", "none", 2)])
def test_run_ahead_equals_single_steps(reorth, basis, m):
    model, p, x, y, (pd, xd, yd) = _case()
    z = si.make_probe(len(p), 0)
    zd = torch.from_numpy(z).cuda()
    ctx = hf.Context(model, 256, m, "f32", basis)
    res = ctx.hf_slq(pd, xd, yd, 256, 1, zd, 1, m, reorth)
    assert ctx.hf_lanczos_iterations() == m
    q_run = torch.empty(ctx.n, device="cuda")
    ctx.hf_lanczos_get_vector(0, q_run)
    ctx.hf_lanczos_init(zd, reorth)
    steps = [ctx.hf_lanczos_step(pd, xd, yd, 256, 1) for _ in range(m)]
    q_step = torch.empty(ctx.n, device="cuda")
    ctx.hf_lanczos_get_vector(0, q_step)
    # nothing in either chain depends on timing: bit for bit the same
    np.testing.assert_array_equal(res["alpha"][0], [s[0] for s in steps])
    np.testing.assert_array_equal(res["beta"][0], [s[1] for s in steps])
    assert torch.equal(q_run, q_step)
    ao, bo, _ = olz.lanczos(lambda q: om.hvp(model, p.astype(np.float64), x, y, q), z.astype(np.float64), m, reorth)
    k = min(m, 6)
    np.testing.assert_allclose(res["alpha"][0][:k], ao[:k], rtol=0, atol=1e-5 * np.abs(ao).max())
    np.testing.assert_allclose(res["beta"][0][:k], bo[:k], rtol=0, atol=1e-5 * np.abs(bo).max())
    ctx.close()


@pytest.mark.parametrize("reorth,basis", [("full", "f32"), ("none", "none")])
def test_run_ahead_stops_at_a_breakdown_and_at_bad_labels(reorth, basis):
    model, p, x, y, (pd, xd, yd) = _case()
    zd = torch.from_numpy(si.make_probe(len(p), 1)).cuda()
    ctx = hf.Context(model, 256, 10, "f32", basis)
    free = ctx.hf_slq(pd, xd, yd, 256, 1, zd, 1, 10, reorth)
    beta = free["beta"][0]
    stop = 4
    tol = float(beta[stop]) * 1.0000001
    expect = next(k for k in range(10) if beta[k] < tol)  # the first iteration below that tolerance
    res = ctx.hf_slq(pd, xd, yd, 256, 1, zd, 1, 10, reorth, tol=tol)
    assert res["status"] == hf.binding.HF_EBREAKDOWN and res["m_eff"][0] == expect + 1 == ctx.hf_lanczos_iterations()
    np.testing.assert_array_equal(res["alpha"][0][:expect + 1], free["alpha"][0][:expect + 1])
    # the vectors and the state left behind are those of single steps: products enqueued ahead of the breakdown change
    # nothing (with a basis q_k's row was not written, on either way)
    def left_behind():
        which = (1, 2) if reorth == "full" else (0, 1, 2)
        vecs = [torch.empty(ctx.n, device="cuda") for _ in which]
        for w, dst in zip(which, vecs):
            ctx.hf_lanczos_get_vector(w, dst)
        state = torch.zeros(ctx.hf_lanczos_state_bytes(), dtype=torch.uint8, device="cuda")
        ctx.hf_lanczos_export(state, state.numel())
        return vecs, state[:128].cpu()   # the header: iterations, end reached, beta_{k-1}
    run_vecs, run_header = left_behind()
    ctx.hf_lanczos_init(zd, reorth)
    statuses = [ctx.hf_lanczos_step(pd, xd, yd, 256, 1, tol)[2] for _ in range(expect + 1)]
    assert statuses[:-1] == [hf.binding.HF_OK] * expect and statuses[-1] == hf.binding.HF_EBREAKDOWN
    step_vecs, step_header = left_behind()
    for a, b in zip(run_vecs, step_vecs):
        assert torch.equal(a, b)
    assert torch.equal(run_header, step_header)
    # two probes, the first of which breaks down: the second starts afresh
    z2 = torch.stack([zd, torch.from_numpy(si.make_probe(len(p), 2)).cuda()])
    both = ctx.hf_slq(pd, xd, yd, 256, 1, z2, 2, 10, reorth, tol=tol)
    assert both["m_eff"][0] == expect + 1
    np.testing.assert_array_equal(both["alpha"][0][:expect + 1], free["alpha"][0][:expect + 1])
    alone = ctx.hf_slq(pd, xd, yd, 256, 1, z2[1], 1, 10, reorth, tol=tol)
    k = alone["m_eff"][0]
    np.testing.assert_array_equal(both["alpha"][1][:k], alone["alpha"][0][:k])
    bad = yd.clone()
    bad[7] = 1000
    with pytest.raises(hf.HessformerError) as e:
        ctx.hf_slq(pd, xd, bad, 256, 1, zd, 1, 10, reorth)
    assert e.value.code == hf.binding.HF_EINVAL
    del e  # its traceback refers to this frame, and the frame to it: the tensors here would outlive the test
    again = ctx.hf_slq(pd, xd, yd, 256, 1, zd, 1, 10, reorth)
    np.testing.assert_array_equal(again["alpha"], free["alpha"])
    ctx.close()


@pytest.mark.parametrize("dtype,vocab", [("f32", 137), ("bf16", 137), ("f32", 138)])
def test_short_and_longer_vectors_take_the_same_steps(dtype, vocab):
    # n = 8192 (the most the one-block update takes) and n = 8216: the same operator family on both sides of the limit,
    # against the oracle; with bf16 parameters the update also leaves the operand-type copies of the rows
    model = si._gpt(1, 24, 2, 32, vocab, 32)
    n = si.num_params(model)
    assert n == (8192 if vocab == 137 else 8216)
    ctx = hf.Context(model, 1, 8, dtype, "f32")
    d = np.random.default_rng(3).uniform(-1, 2, n).astype(np.float32)
    z = si.make_probe(n, 3)
    dd = torch.from_numpy(d).cuda()
    q = torch.empty(n, device="cuda")
    ctx.hf_lanczos_init(torch.from_numpy(z).cuda(), "full")
    al, be = [], []
    for _ in range(8):
        ctx.hf_lanczos_get_vector(0, q)
        a, b, _ = ctx.hf_lanczos_update(dd * q)
        al.append(a)
        be.append(b)
    ao, bo, _ = olz.lanczos(lambda u: d.astype(np.float64) * u, z.astype(np.float64), 8, "full")
    np.testing.assert_allclose(al, ao, rtol=1e-5, atol=1e-5)
    np.testing.assert_allclose(be, bo, rtol=1e-5, atol=1e-5)
    ctx.close()
