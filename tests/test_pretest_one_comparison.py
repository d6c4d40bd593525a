"""The main pass's float32 test in the form of one comparison, e < max(rest, 0)^2, with the sums of a column's rows formed in
pairs: replayed in numpy float32 on the windows of test_pretest_bounds and compared with exact arithmetic.  (The
constants are typed in here, and compared with those of the kernel source; test_pretest_bounds runs that source itself.)"""
import re

import numpy as np
import pytest

from tests import test_pretest_bounds as bounds

f32 = np.float32


def _round_up32(x):
    y = f32(x)
    return np.nextafter(y, f32(np.inf)) if float(y) < x else y


def _column(r, P):
    """Window sum of the row sums r[:, 0 .. P - 1], in the kernel's order."""
    add = lambda a, b: (a + b).astype(f32)
    pair = lambda i: add(r[:, i - 1], r[:, i])
    if P == 1:
        return r[:, 0]
    if P == 3:
        return add(r[:, 0], pair(2))
    if P == 5:
        return add(add(pair(1), pair(3)), r[:, 4])
    return add(add(add(pair(1), pair(3)), pair(5)), r[:, 6])


def _kept(P, alpha, W, bound, slack=1.3, extra=2e-6, bound_terms=2.04):
    n = P * P
    ca, cb = alpha / n, (1.0 - alpha) / n
    kslack = float(f32(f32(slack) * f32(3.0 * n + 3.0) * f32(bounds.U)))
    caf, cbf, a = f32(ca), f32(cb), _round_up32(cb * cb * n * (1.0 + kslack) * (1.0 + extra))
    bound_lof = bounds._round_down32(bound.astype(np.float64) * (1.0 - 2.0 ** -22 - bound_terms * n * bounds.U))
    ra, rs, rq = np.abs(W[:, :, 0]), W[:, :, 0].copy(), (W[:, :, 0] * W[:, :, 0]).astype(f32)
    for j in range(1, P):
        ra = (ra + np.abs(W[:, :, j])).astype(f32)
        rs = (rs + W[:, :, j]).astype(f32)
        rq = bounds._fma32(W[:, :, j], W[:, :, j], rq)
    sa, ss, sq = _column(ra, P), _column(rs, P), _column(rq, P)
    with np.errstate(all="ignore"):
        m = (cbf * ss).astype(f32)
        e = bounds._fma32(-m, m, (a * sq).astype(f32))
        t = np.fmax(bounds._fma32(np.full_like(sa, -caf), sa, bound_lof), f32(0))
        return ~(e < (t * t).astype(f32))


def test_the_constants_are_the_sources():
    """... and the replay gives what the source's code gives, window by window."""
    pre = bounds._piece(open(bounds.SOURCE).read(), "template <int P> struct PreF32 {", "\n};")
    assert re.search(r"kSlack = ([\d.]+)f \* \(3\.f \* P \* P \+ 3\.f\) \* ([\d.e-]+)f;", pre).groups() == ("1.3", "5.9604645e-8")
    assert re.search(r"kBoundFactor = 1\.0 - 1\.0 / (\d+)\.0 - ([\d.]+) \* \(P \* P\) \* ([\d.e-]+);", pre).groups() == (str(2 ** 22), "2.04", "5.9604645e-8")
    assert "* (1.0 + static_cast<double>(kSlack)) * (1.0 + 2e-6))" in pre
    rng = np.random.default_rng(1)
    for P in (3, 5, 7):
        for name, W in bounds._windows(rng, P, 2000).items():
            b = np.abs(W).mean(axis=(1, 2)).astype(f32) * rng.uniform(0.5, 2.0, len(W)).astype(f32)
            assert np.array_equal(_kept(P, 0.5, W, b), bounds._kept(P, 0.5, W, b)), (P, name)


@pytest.mark.parametrize("P", [1, 3, 5, 7])
def test_no_centre_that_reaches_the_bound_is_ruled_out(P, monkeypatch):
    monkeypatch.setattr(bounds, "_kept", _kept)
    wrong, clear, kept_clear = bounds._sweep(P, seed=300 + P, N=6000)
    assert wrong == 0
    assert clear > 5000 and kept_clear == 0


@pytest.mark.parametrize("P", [3, 7])
def test_without_the_slacks_centres_are_lost(P, monkeypatch):
    monkeypatch.setattr(bounds, "_kept", _kept)
    wrong, _, _ = bounds._sweep(P, seed=400 + P, N=3000, slack=0.0, extra=0.0, bound_terms=0.0)
    assert wrong > 100


def test_values_that_are_not_numbers_keep_the_centre():
    W = np.full((3, 3, 3), 1e-3, f32)
    W[0, 1, 1], W[1, 0, 2], W[2, 2, 2] = np.nan, np.inf, -np.inf
    for alpha in (0.0, 0.5, 1.0):
        assert _kept(3, alpha, W, np.full(3, 1.0, f32)).all()
