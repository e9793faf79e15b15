"""The decision of the first orthogonalisation pass whether it may write q_{k+1} itself (over q_{k-1}, with a bf16 basis): never where beta_k turns out
below the tolerance, however the rows lie to each other, and as a rule in the runs that it is there for.  Host code only."""
import ctypes

import numpy as np
import pytest

import paper_2505_11564_amd as hf


def _plan(Q, w, tol):
    """(before, est) for float64 rows Q (q_k last), as the kernel's sums give them."""
    c = Q @ w
    old = c[:-2] if len(c) > 1 else c[:0]
    qk, qp = Q[-1], Q[-2] if len(c) > 1 else np.zeros_like(Q[-1])
    s = [c[-1], qp @ w, w @ w, old @ old, np.abs(old).sum(), (old**2).max() if len(old) else 0.0, qk @ qk, qp @ qp, qk @ qp, tol]
    out = (ctypes.c_double * 2)()
    hf.lib().hf_internal_lz_first_plan((ctypes.c_double * 10)(*s), out)
    return out[0], out[1]


def _rows(rng, n, k, most):
    """k orthonormal rows, and the older ones again with every element moved by up to `most` of itself (2^-9: rounded to bf16) towards or away from
    a common direction, the worst that rounding may do."""
    q, _ = np.linalg.qr(rng.standard_normal((n, k + 1)))
    q, u = q[:, :k].T.copy(), q[:, k]
    rounded = q.copy()
    for j in range(k - 2):
        rounded[j] *= 1.0 + most * np.sign(q[j] * (q[-1] + 0.5 * q[-2])) * rng.choice([-1, 1])
    return rounded, u


@pytest.mark.parametrize("n,k", [(12, 4), (40, 3), (40, 6), (300, 9), (300, 40)])
def test_nothing_is_written_early_below_the_tolerance(n, k):
    rng = np.random.default_rng(n + k)
    early = 0
    for trial in range(300):
        Q, u = _rows(rng, n, k, 2.0**-9)
        c = np.zeros(k)
        c[-1], c[-2] = rng.standard_normal(2) * rng.choice([1.0, 0.1, 3.0], 2)
        c[:-2] = rng.standard_normal(k - 2) * 10.0 ** rng.uniform(-6, -0.5)
        beta = np.linalg.norm(c) * 10.0 ** rng.uniform(-1.55, 0.5)
        w = Q.T @ c + beta * u
        true = np.linalg.norm(w - Q.T @ (Q @ w))
        for f in (1.0 + 1e-9, 1.01, 1.2):
            assert _plan(Q, w, true * f)[1] == 0.0
        early += _plan(Q, w, 0.9 * true)[1] > 0.0
        est = _plan(Q, w, 0.0)[1]
        assert est == 0.0 or abs(est - true) <= 0.3 * true
    assert early > 30


@pytest.mark.parametrize("n,k", [(300, 1), (300, 2), (300, 9), (10608, 40)])
def test_a_run_writes_early(n, k):
    """alpha, beta and beta_{k-1} of one size; older coefficients at the level that rounding leaves."""
    rng = np.random.default_rng(k)
    q, _ = np.linalg.qr(rng.standard_normal((n, k + 1)))
    Q, u = q[:, :k].T, q[:, k]
    c = rng.uniform(0.4, 0.6, k)
    c[:-2] = 2.0**-9 / n**0.5 * rng.standard_normal(max(0, k - 2))
    w = Q.T @ c + 0.5 * u
    for tol in (0.0, 0.49):
        before, est = _plan(Q, w, tol)
        assert abs(est - 0.5) <= 1e-6 and abs(before - np.hypot(0.5, np.linalg.norm(c[:-2]))) <= 1e-6
    assert _plan(Q, w, 0.4999)[1] == 0.0 and _plan(Q, w, 0.6)[1] == 0.0
    assert _plan(Q, np.full(n, np.nan), 0.0)[1] == 0.0 and _plan(Q, np.zeros(n), 0.0)[1] == 0.0
    assert _plan(Q, Q.T @ c + 1e-4 * u, 0.0) == (np.inf, 0.0)   # the difference has lost its digits
