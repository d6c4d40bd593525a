"""The float32 test with which the main pass rules out centres below a layer's candidate bound
(before the evaluation in full): the device code itself (the sums of rows and columns, the factors with their slacks, the
comparison), taken from the kernel source, compiled for the CPU and run on hard windows, against exact
arithmetic: no centre whose exact score reaches the bound is ever ruled out; with the slacks taken out of the source, many are.
Sides 3, 5 and 7: single elements have no such test.
NSI of a window: alpha * mean|w| + (1 - alpha) * std w (Eqs. 8-10)."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

f32 = np.float32
U = 5.9604645e-8          # 2^-24
SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_17530_amd", "csrc", "rsdgc_kernels.hip")

_SHIM = r"""
#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ inline
static float __double2float_rd(double x) { const float y = (float)x; return (double)y > x ? std::nextafterf(y, -INFINITY) : y; }
static float __double2float_ru(double x) { const float y = (float)x; return (double)y < x ? std::nextafterf(y, INFINITY) : y; }
"""
_KEPT = r"""
template <int P> static void kept_p(double alpha, const float *w, const float *bound, long n, unsigned char *out) {
    const double ca = alpha / (P * P), cb = (1.0 - alpha) / (P * P);
    const float a = PreF32<P>::square_factor(cb);
    for (long k = 0; k < n; ++k, w += P * P) {
        ColumnSums<P> sa, ss, sq;
        for (int i = 0; i < P; ++i) {
            float ra, rs, rq;
            row_sums<P>(w + i * P, ra, rs, rq);
            sa.push(i, ra);
            ss.push(i, rs);
            sq.push(i, rq);
        }
        out[k] = PreF32<P>::stays(sa.window(P - 1), ss.window(P - 1), sq.window(P - 1), (float)ca, (float)cb, a, PreF32<P>::bound(bound[k]));
    }
}
extern "C" void kept(int p, double alpha, const float *w, const float *bound, long n, unsigned char *out) {
    p == 3 ? kept_p<3>(alpha, w, bound, n, out) : p == 5 ? kept_p<5>(alpha, w, bound, n, out) : kept_p<7>(alpha, w, bound, n, out);
}
"""


def _piece(src, start, end):
    i = src.index(start)
    assert src.count(start) == 1
    return src[i:src.index(end, i) + len(end)] + "\n"


@functools.lru_cache(maxsize=None)
def _compiled(slacks):
    """The library with the source's code; slacks False: its three slacks set to 0."""
    src = open(SOURCE).read()
    code = (_piece(src, "template <int P> struct PreF32 {", "\n};") +
            _piece(src, "template <int P>\n__device__ __forceinline__ void row_sums(", "\n}") +
            _piece(src, "template <int P>\nstruct ColumnSums {", "\n};"))
    if not slacks:
        for text, without in (("1.3f * (3.f", "0.f * (3.f"), ("(1.0 + 2e-6)", "1.0"), ("2.04 * (P * P)", "0.0 * (P * P)")):
            assert code.count(text) == 1
            code = code.replace(text, without)
    folder = tempfile.mkdtemp()
    try:
        with open(os.path.join(folder, "pre.cpp"), "w") as f:
            f.write(_SHIM + code + _KEPT)
        lib = os.path.join(folder, "pre.so")
        subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", os.path.join(folder, "pre.cpp"), "-o", lib], check=True)
        return ctypes.CDLL(lib)
    finally:
        shutil.rmtree(folder, ignore_errors=True)


def _fma32(a, b, c):
    # round32(a * b + c): the product of two float32 is exact in double
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(f32)


def _round_down32(x):
    y = x.astype(f32)
    return np.where(y.astype(np.float64) > x, np.nextafter(y, f32(-np.inf)), y).astype(f32)


def _kept(P, alpha, W, bound, slacks=True):
    """The test as the main pass applies it: True where the centre stays (queued for evaluation)."""
    W, bound, out = np.ascontiguousarray(W, f32), np.ascontiguousarray(bound, f32), np.zeros(len(W), np.uint8)
    ptr = lambda x: ctypes.c_void_p(x.ctypes.data)
    _compiled(slacks).kept(ctypes.c_int(P), ctypes.c_double(alpha), ptr(W), ptr(bound), ctypes.c_long(len(W)), ptr(out))
    return out.astype(bool)


def _must_stay(P, alpha, W, bound):
    """Exact: the score reaches what rounds to the bound in float32 (with the evaluation's own 1e-9)."""
    n = P * P
    Wd = W.astype(np.longdouble)
    SA, SS, SQ = np.abs(Wd).sum(axis=(1, 2)), Wd.sum(axis=(1, 2)), (Wd * Wd).sum(axis=(1, 2))
    D = np.maximum(n * SQ - SS * SS, 0)
    S = np.longdouble(alpha / n) * SA + np.longdouble((1.0 - alpha) / n) * np.sqrt(D)
    return S >= bound.astype(np.longdouble) * (np.longdouble(1) - np.longdouble(2.0) ** -22)


def _windows(rng, P, N):
    n = P * P
    c = rng.standard_normal((N, 1, 1)).astype(f32)
    one_large = rng.standard_normal((N, P, P)).astype(f32) * f32(1e-4)
    one_large[:, 0, 0] = rng.standard_normal(N).astype(f32)
    signs = np.where((np.arange(n).reshape(P, P) % 2) == 0, 1, -1).astype(f32)
    return {
        "noise": rng.standard_normal((N, P, P)).astype(f32),
        "near-constant": (c * (1 + rng.integers(-4, 5, (N, P, P)) * 2.0 ** -23)).astype(f32),
        "constant": np.broadcast_to(c, (N, P, P)).astype(f32).copy(),
        "one large value": one_large,
        "alternating signs": np.abs(rng.standard_normal((N, P, P))).astype(f32) * signs,
        "six decades": (rng.standard_normal((N, P, P)) * 10.0 ** rng.uniform(-6, 0, (N, P, P))).astype(f32),
        "ramp on an offset": (c * (1 + np.arange(n).reshape(1, P, P) * 2.0 ** -20)).astype(f32),
    }


def _sweep(P, seed, N, **kw):
    rng = np.random.default_rng(seed)
    n = P * P
    wrong = clear = kept_clear = 0      # clear: noise windows whose score lies 10 % below the bound
    for alpha in (0.5, 0.0, 1.0, 0.25, 0.9):
        for name, W in _windows(rng, P, N).items():
            for scale in (1.0, 2.0 ** -38, 2.0 ** 38, 1e-3):
                Ws = (W * f32(scale)).astype(f32)
                Wd = Ws.astype(np.float64)
                SA, SS, SQ = np.abs(Wd).sum(axis=(1, 2)), Wd.sum(axis=(1, 2)), (Wd * Wd).sum(axis=(1, 2))
                S = alpha / n * SA + (1 - alpha) / n * np.sqrt(np.maximum(n * SQ - SS * SS, 0))
                # bounds right at the score, a hair to either side, and well away from it
                eps = rng.choice([0.0, 1e-8, -1e-8, 1e-7, -1e-7, 3e-7, -3e-7, 1e-6, -1e-6, 1e-5, 1e-3, -1e-3, 0.1, -0.1], size=N)
                b = (S * (1 + eps)).astype(f32)
                ok = np.isfinite(b) & (b >= 2.0 ** -40) & (b <= 2.0 ** 40)     # the range bounds are handed out in
                if not ok.any():
                    continue
                kept, must = _kept(P, alpha, Ws[ok], b[ok], **kw), _must_stay(P, alpha, Ws[ok], b[ok])
                wrong += int((must & ~kept).sum())
                if name == "noise":
                    far = eps[ok] >= 0.1
                    clear += int(far.sum())
                    kept_clear += int((kept & far).sum())
    return wrong, clear, kept_clear


@pytest.mark.parametrize("P", [3, 5, 7])
def test_no_centre_that_reaches_the_bound_is_ruled_out(P):
    wrong, clear, kept_clear = _sweep(P, seed=100 + P, N=6000)
    assert wrong == 0
    assert clear > 5000 and kept_clear == 0      # and what lies clearly below the bound is still ruled out


@pytest.mark.parametrize("P", [3, 7])
def test_without_the_slacks_centres_are_lost(P):
    """The same code with the slack on the squares and the extra terms of the bound's factor taken out: the
    sweep above has the power to see a bound that is too tight."""
    wrong, _, _ = _sweep(P, seed=200 + P, N=3000, slacks=False)
    assert wrong > 100
