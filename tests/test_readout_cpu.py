"""hf_tridiag_readout on tridiagonal matrices that are hard for an iteration with shifts: blocks that fall apart, graded and huge and denormal entries,
close eigenvalues.  Against numpy's symmetric solver; 3e-14 of the norm is some hundred roundings of its float64 (measured up to 8e-15)."""
import numpy as np
import pytest

import paper_2505_11564_amd as hf


def _matrix(kind, k):
    rng = np.random.default_rng(k)
    one, a = np.ones(k), rng.standard_normal(k)
    if kind == "random":
        return a, np.abs(rng.standard_normal(k))
    if kind == "zero_diagonal":
        return 0 * one, one
    if kind == "close_pairs":
        return np.abs(np.arange(k) - (k - 1) / 2), one
    if kind == "graded_down":
        return 10.0 ** -np.linspace(0, 300, k), 10.0 ** -np.linspace(0, 300, k)
    if kind == "graded_up":
        return 10.0 ** np.linspace(-300, 0, k), 10.0 ** np.linspace(-300, 0, k)
    if kind == "blocks":
        return a, np.where(np.arange(k) % 3 == 1, 0.0, 1.0)
    if kind == "diagonal":
        return a, 0 * one
    if kind == "multiple":
        return one, 1e-18 * one
    if kind == "huge":
        return 2.5e307 * one, 1e307 * one
    return 0 * one, 5e-324 * one  # denormal


@pytest.mark.parametrize("k", [1, 2, 3, 7, 50, 300])
@pytest.mark.parametrize("kind", ["random", "zero_diagonal", "close_pairs", "graded_down", "graded_up", "blocks", "diagonal", "multiple", "huge", "denormal"])
def test_readout(kind, k):
    a, b = _matrix(kind, k)
    want = np.linalg.eigvalsh(np.diag(a) + np.diag(b[:k - 1], 1) + np.diag(b[:k - 1], -1))
    ritz, w, last = hf.hf_tridiag_readout(a, b, want_last_row=True)
    norm = max(np.abs(want).max(), 1e-300)
    assert np.all(np.diff(ritz) >= 0) and np.all(w >= 0)
    assert np.abs(ritz - want).max() <= 3e-14 * norm
    # both rows are unit vectors, and T's corner elements come back from them
    for weights, corner in ((w, a[0]), (last**2, a[-1])):
        assert abs(weights.sum() - 1) <= 3e-14
        assert abs((weights * ritz).sum() - corner) <= 3e-14 * norm


def test_readout_of_what_is_not_finite():
    for bad in (np.nan, np.inf):
        for a, b in (([1.0, bad], [1.0, 1.0]), ([1.0, 2.0, 3.0], [bad, 1.0, 1.0])):
            ritz, w, last = hf.hf_tridiag_readout(a, b, want_last_row=True)
            assert np.isnan(ritz).all() and np.isnan(w).all() and np.isnan(last).all()
