"""The accumulators of the exact backprojection, run on the CPU, against
Python's integers: no bit of any partial sum is lost at any scale the walk can
give, whatever the signs and the order, and the conversion to float64 is within
two roundings of the exact value."""

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


@pytest.fixture(scope="module")
def lib():
    os.makedirs(BUILD, exist_ok=True)
    out, src = os.path.join(BUILD, "libexact_sums_probe.so"), os.path.join(HERE, "exact_sums_probe.cpp")
    if not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(f) for f in
                                                              (src, os.path.join(CSRC, "kernels.h"))):
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "-O2",
                        "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-gpu-rdc",
                        "-Wno-unused-command-line-argument", "-I", CSRC, "-I", os.path.join(ROOT, "include"), src,
                        "-o", out + ".tmp"], check=True, capture_output=True)
        os.replace(out + ".tmp", out)
    L = C.CDLL(out)
    L.probe_sum.restype = C.c_double
    L.probe_digit_bits.argtypes = [C.c_longlong]
    return L


@pytest.mark.parametrize("rays", [1, 2 ** 26, 2 ** 26 + 1, 94371840, 2 ** 33, 2 ** 40])
@pytest.mark.parametrize("kind", ["one scale", "all scales", "extremes", "cancelling"])
def test_sums_are_exact(lib, rays, kind):
    bits = lib.probe_digit_bits(rays)
    words = lib.probe_words(bits)
    # a word holds one digit below 2^(bits - 1) from every ray
    assert (bits - 1) + int(np.ceil(np.log2(rays))) <= 62
    rng = np.random.default_rng(int(np.log2(rays)) * 7 + len(kind))
    n = 500
    m = rng.integers(-2 ** 57 + 1, 2 ** 57, size=n)
    scale = rng.integers(-78, 121, size=n)
    if kind == "one scale":
        scale[:] = 37
    elif kind == "extremes":
        scale = rng.choice([-78, -77, 119, 120], size=n)
        m = rng.choice([-2 ** 57 + 1, -1, 1, 2 ** 57 - 1], size=n)
    elif kind == "cancelling":
        m[n // 2:], scale[n // 2:] = -m[: n // 2], scale[: n // 2]
        m[-1] += 1
    w = np.zeros(words, np.uint64)
    scale, m = scale.astype(np.int32), m.astype(np.int64)
    got = lib.probe_sum(bits, C.c_longlong(n), C.c_void_p(scale.ctypes.data), C.c_void_p(m.ctypes.data),
                        C.c_void_p(w.ctypes.data))
    want = sum(Fraction(int(a)) * Fraction(2) ** (-int(s)) for a, s in zip(m, scale))
    held = sum(int(v) * 2 ** (bits * k) for k, v in enumerate(w.astype(np.int64)))
    assert Fraction(held) / 2 ** 120 == want
    assert abs(Fraction(got) - want) <= abs(want) * Fraction(2, 2 ** 52)
    # the other order
    w2 = np.zeros(words, np.uint64)
    scale, m = scale[::-1].copy(), m[::-1].copy()
    lib.probe_sum(bits, C.c_longlong(n), C.c_void_p(scale.ctypes.data), C.c_void_p(m.ctypes.data),
                  C.c_void_p(w2.ctypes.data))
    assert np.array_equal(w, w2)
