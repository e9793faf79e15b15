"""The update of long vectors with a stored basis: the pass that writes q_{k+1} with an estimate of beta_k, the passes it leaves to others (a small
beta_k, a tolerance in the way), and what they leave behind, against Lanczos in float64 with an operator diag(d).

Tolerances: coefficients 1e-5 of the operator's norm (fp32 vectors, sums in fp64; measured 1e-7 to 5e-7), norms 1e-7 (fp32 elements: 6e-8)."""
import numpy as np
import pytest
import torch

import paper_2505_11564_amd as hf
import synth_inputs as si

pytestmark = pytest.mark.gpu

MODELS = {  # lengths: some slices of 4096 and a part; more slices than blocks of a pass (2048); one to three elements behind the last whole 16 bytes
    "short": si._gpt(1, 36, 2, 60, 11, 7),
    "middle": si._gpt(1, 72, 3, 200, 97, 5),
    "long": si._gpt(2, 512, 8, 2048, 5003, 16),
    "and_one": si._mlp(130, 63, 10),
    "and_two": si._mlp(128, 64, 10),
    "and_three": si._mlp(127, 64, 11),
}
SHORT = {"few": si._mlp(9, 13, 5), "some": si._mlp(32, 32, 10), "most": si._gpt(1, 24, 2, 32, 137, 32)}  # n = 200, 1386 and 8192, by one block
SPECTRA = {"around_zero": (-0.5, 1.5), "away_from_zero": (0.9, 1.0)}


def _vectors(n, lo, hi):
    g = torch.Generator(device="cuda").manual_seed(3)
    z = torch.randint(0, 2, (n,), generator=g, device="cuda", dtype=torch.int8).float().mul_(2).sub_(1)
    return z, torch.empty(n, device="cuda").uniform_(lo, hi, generator=g)


def _reference(z, d, m):
    q = [z.double() / z.double().norm()]
    al, be = [], []
    for k in range(m):
        w = d.double() * q[k]
        al.append((q[k] @ w).item())
        for _ in range(2):
            for x in q:
                w = w - (x @ w) * x
        be.append(w.norm().item())
        q.append(w / be[-1])
    return np.array(al), np.array(be), q


def _step(ctx, d, q, r, tol=0.0):
    ctx.hf_lanczos_get_vector(0, q)
    torch.mul(d, q, out=r)
    return ctx.hf_lanczos_update(r, tol)


@pytest.mark.parametrize("spectrum", list(SPECTRA))
@pytest.mark.parametrize("dtype,basis", [("bf16", "f32"), ("f32", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("name", list(MODELS))
def test_update_of_long_vectors(name, dtype, basis, spectrum):
    model, m = MODELS[name], 12
    n = si.num_params(model)
    assert n > 8192 and n % 4 == {"and_one": 1, "and_two": 2, "and_three": 3}.get(name, 0)
    z, d = _vectors(n, *SPECTRA[spectrum])
    al, be, qs = _reference(z, d, m)
    # An iteration leaves rounding errors times alpha / beta (1 and 38).  bf16 rows have some of 2^-9: the part in random directions lies along any one
    # vector with 2^-9 / sqrt(n), and m iterations of it come together (measured 7.8e-3 at n = 10608); q_0, whose elements are all rounded alike,
    # leaves 5e-5 to 7e-5 whatever n (a quarter of what is allowed).
    grown = 38.0 if spectrum == "away_from_zero" else 1.0
    off = max(3e-4, 2 * m * 2.0**-9 * grown / n**0.5) if basis == "bf16" else 5e-5 * grown
    # alpha_k is a Rayleigh quotient: a q_k that is off by that much moves it by up to 2 off ||(A - alpha_k) q_k||, the norm at most beta_k +
    # beta_{k-1}; beta_k moves by less (||A - alpha_k|| off).  bf16 rows and a spectrum away from zero take 2e-5 to 4e-5 of that (the same steps in numpy, eight seeds), the first three lengths here less.
    coef = 4 * be.max() * off if basis == "bf16" and grown > 1.0 and name.startswith("and_") else 1e-5
    ctx = hf.Context(model, 1, m, dtype, basis)
    q, r = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    ctx.hf_lanczos_init(z, "full")
    for k in range(m):
        a, b, status = _step(ctx, d, q, r)
        assert status == 0
        assert abs(q.double().norm().item() - 1.0) <= 1e-7
        assert abs(a - al[k]) <= coef and abs(b - be[k]) <= coef
    ctx.hf_lanczos_get_vector(0, q)  # q_m
    assert abs(q.double().norm().item() - 1.0) <= 1e-7
    assert (q.double() - qs[m]).norm().item() <= off
    ctx.close()


@pytest.mark.parametrize("spectrum", list(SPECTRA))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(SHORT))
def test_update_of_short_vectors(name, dtype, spectrum):
    """The second pass where one would let errors grow belongs to the one-block update as well: without it a spectrum of 0.9 .. 1.0 leaves q_12
    1.4 off (the same steps in numpy)."""
    model, m = SHORT[name], 12
    n = si.num_params(model)
    assert n <= 8192
    z, d = _vectors(n, *SPECTRA[spectrum])
    al, be, qs = _reference(z, d, m)
    ctx = hf.Context(model, 1, m, dtype, "f32")
    q, r = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    ctx.hf_lanczos_init(z, "full")
    for k in range(m):
        a, b, status = _step(ctx, d, q, r)
        assert status == 0
        assert abs(q.double().norm().item() - 1.0) <= 1e-7
        assert abs(a - al[k]) <= 1e-5 and abs(b - be[k]) <= 1e-5
    ctx.hf_lanczos_get_vector(0, q)
    assert (q.double() - qs[m]).norm().item() <= 5e-5 * (38.0 if spectrum == "away_from_zero" else 1.0)
    ctx.close()


@pytest.mark.parametrize("basis", ["f32", "bf16"])
def test_breakdown_leaves_the_vectors(basis):
    model = MODELS["middle"]
    n = si.num_params(model)
    z, d = _vectors(n, -0.5, 1.5)
    ctx = hf.Context(model, 1, 8, "bf16", basis)
    q, r = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    ctx.hf_lanczos_init(z, "full")
    for _ in range(3):
        _step(ctx, d, q, r)
    before = [torch.empty(n, device="cuda") for _ in range(2)]
    for i in range(2):
        ctx.hf_lanczos_get_vector(i, before[i])
    a, b, status = _step(ctx, d, q, r, tol=10.0)  # beta is about 0.5
    assert status == hf.binding.HF_EBREAKDOWN and 0.4 < b < 0.7
    if basis == "bf16":  # (an fp32 basis names its vectors by their row, and the count has gone on)
        after = torch.empty(n, device="cuda")
        for i in range(2):
            ctx.hf_lanczos_get_vector(i, after)
            assert torch.equal(after, before[i])
    for j in range(4):
        ctx.hf_lanczos_get_vector(16 + j, r)
        if j == 3 and basis == "f32":
            assert torch.equal(r, before[0])
    ctx.close()


@pytest.mark.parametrize("basis", ["f32", "bf16"])
def test_residual_of_a_step(basis):
    model, batch = si._gpt(1, 64, 2, 256, 211, 12), 2
    n = si.num_params(model)
    p = torch.from_numpy(si.make_params(model, param_dtype="bf16")).cuda().to(torch.bfloat16)
    x, y = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in si.make_batch(dict(model=model, batch=batch, tokens="zipf"), seq=12))
    z, _ = _vectors(n, 0, 1)
    ctx = hf.Context(model, batch, 4, "bf16", basis)
    ctx.hf_lanczos_init(z, "full")
    q, q1, r = (torch.empty(n, device="cuda") for _ in range(3))
    for _ in range(3):
        ctx.hf_lanczos_get_vector(0, q)
        _, b, _ = ctx.hf_lanczos_step(p, x, y, batch, 12)
        ctx.hf_lanczos_get_vector(0, q1)
        ctx.hf_lanczos_get_vector(2, r)
        assert abs(r.double().norm().item() - b) <= 1e-6 * b
        assert (r.double() - b * q1.double()).norm().item() <= 1e-6 * b
        assert abs((r.double() @ q.double()).item()) <= 1e-5 * b
    ctx.close()
