"""The exact determinant signs behind the walk's filters, run on the CPU,
against rational arithmetic.

Columns whose scaled entries are integers below 2^42 are decided in integers of
30-bit digits, all others by the floating-point expansion; both must give the
sign of the exact determinant, and the two must agree wherever both apply.
The inputs sit where the integer route can go wrong: exact zeros and their
nearest neighbours, entries as large as the route admits in all nine places
(the largest determinants), columns just inside and just outside of it,
denormal, huge and zero columns, absent points, infinities and NaN (which
must never take it).
"""

import ctypes as C
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1908_06909_amd", "csrc")
BUILD = os.path.join(ROOT, "_build")
f32 = np.float32


@pytest.fixture(scope="module")
def probe():
    os.makedirs(BUILD, exist_ok=True)
    out, src = os.path.join(BUILD, "libexact_probe.so"), os.path.join(HERE, "exact_probe.cpp")
    if not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(f) for f in
                                                              (src, os.path.join(CSRC, "exact.h"))):
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "-O2",
                        "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-fast-math", "-fno-gpu-rdc",
                        "-Wno-unused-command-line-argument", "-I", CSRC, src, "-o", out + ".tmp"],
                       check=True, capture_output=True)
        os.replace(out + ".tmp", out)
    lib = C.CDLL(out)

    def run(pts, null=None):
        pts = np.ascontiguousarray(pts, f32).reshape(-1, 6, 3)
        n = len(pts)
        null = np.zeros((n, 6), np.int32) if null is None else np.ascontiguousarray(null, np.int32)
        res = [np.zeros(n, np.int32) for _ in range(3)]
        lib.probe_exact(C.c_longlong(n), *(C.c_void_p(a.ctypes.data) for a in (pts, null, *res)))
        return pts, null, res

    return run


def _reference(pts, null):
    p = [[Fraction(0)] * 3 if null[i] else [Fraction(float(v)) for v in pts[i]] for i in range(6)]
    a, b, c = ([p[2 * k][i] - p[2 * k + 1][i] for i in range(3)] for k in range(3))
    d = (a[0] * (b[1] * c[2] - b[2] * c[1]) + a[1] * (b[2] * c[0] - b[0] * c[2])
         + a[2] * (b[0] * c[1] - b[1] * c[0]))
    return (d > 0) - (d < 0)


def _cases(kind, rng, n=400):
    """Points [n, 6, 3] and the route they have to take (1 integer, 0 expansion, None either)."""
    if kind == "mesh":  # nodes of a grid seen from a source: mostly coplanar
        g = rng.integers(-32, 33, size=(n, 6, 3)) / 64.0
        g[:, 1::2] = np.array([4.0, 0.0, 0.0])
        return g, 1
    if kind == "zero and next":  # the third column in the span of the others, and one ulp beside it
        a, b = rng.integers(-2 ** 9, 2 ** 9, size=(2, n, 3))
        c = a * rng.integers(-40, 41, (n, 1)) + b * rng.integers(-40, 41, (n, 1))
        p = np.zeros((n, 6, 3))
        p[:, 0], p[:, 2], p[:, 4] = a, b, c
        p[::2, 4, 0] = np.nextafter(p[::2, 4, 0].astype(f32), f32(np.inf))
        return p, None
    if kind == "largest":  # differences of 2^41 units in every place, signs at random
        p = np.zeros((n, 6, 3))
        s = rng.choice([-1.0, 1.0], size=(n, 3, 3))
        p[:, 0::2], p[:, 1::2] = s * 2.0 ** 40, -s * (2.0 ** 40 - 2.0 ** 16 * rng.integers(0, 4, size=(n, 3, 3)))
        p[:, 0, 0] += 0  # a unit of 1 keeps the columns at the route's largest scale
        return p, 1
    if kind in ("inside", "outside"):  # the smallest unit 2^-40 (2^-42) of the largest entry's power of two
        p = rng.integers(1, 2 ** 20, size=(n, 6, 3)).astype(np.float64) * 2.0 ** -20
        p[:, 1::2] = 0.0
        p[:, 0::2, 0] = 0.5 + p[:, 0::2, 0] / 4
        bits = 41 if kind == "inside" else 43
        p[:, 0::2, 1] = (2 * rng.integers(1, 2 ** 10, size=(n, 3)) + 1) * 2.0 ** -bits
        return p, 1 if kind == "inside" else 0
    if kind == "extremes":  # denormal to huge
        e = rng.integers(-149, 127, size=(n, 6, 3)).astype(np.float64)
        return rng.choice([-1.0, 0.0, 1.0], size=(n, 6, 3)) * 2.0 ** e, None
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["mesh", "zero and next", "largest", "inside", "outside", "extremes"])
def test_exact_sign_equals_rational_arithmetic(probe, kind):
    pts, route = _cases(kind, np.random.default_rng(7))
    pts, null, (sign, ints, slow) = probe(pts)
    want = [_reference(p, z) for p, z in zip(pts, null)]
    assert np.array_equal(sign, want)
    assert np.array_equal(slow, want)
    if route is not None:
        assert np.all(ints == route)
    assert kind in ("outside", "extremes") or ints.any()


def test_absent_points_and_zero_columns(probe):
    rng = np.random.default_rng(8)
    pts = rng.integers(-8, 9, size=(200, 6, 3)) / 16.0
    pts[::5, 2:4] = pts[::5, 2:3]  # a zero column
    null = np.zeros((200, 6), np.int32)
    null[:, 3] = 1  # B0 absent, as for the tie rule's axes
    null[::7, 1] = 1
    pts, null, (sign, ints, slow) = probe(pts, null)
    want = [_reference(p, z) for p, z in zip(pts, null)]
    assert np.array_equal(sign, want) and np.array_equal(slow, want) and np.all(ints == 1)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_without_an_integer_never_take_the_integer_route(probe, bad):
    pts = np.tile(np.linspace(-1, 1, 18).reshape(1, 6, 3), (18, 1, 1))
    pts.reshape(18, 18)[np.arange(18), np.arange(18)] = bad
    assert not probe(pts)[2][1].any()
