"""The walk step's first test, one bound from the longest edge of the whole
mesh, on the adversarial walk states of the sign filters' tests: whenever it
calls the three signs certain they are the exact ones, for meshes whose longest
edge is the step's own (the tightest bound there is) and for longer ones."""

import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from test_walk_filter_cpu import BUILD, HERE, ROOT, _exact_step, adversarial_steps, base_steps


@pytest.fixture(scope="module")
def lib():
    os.makedirs(BUILD, exist_ok=True)
    out, src = os.path.join(BUILD, "libstep_bound_probe.so"), os.path.join(HERE, "step_bound_probe.cpp")
    csrc = os.path.join(ROOT, "paper_1908_06909_amd", "csrc")
    if not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(f) for f in
                                                              (src, os.path.join(csrc, "walk_filter.h"))):
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "-O2",
                        "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-fast-math", "-fno-gpu-rdc",
                        "-Wno-unused-command-line-argument", "-I", csrc, "-I", os.path.join(ROOT, "include"), src,
                        "-o", out + ".tmp"], check=True, capture_output=True)
        os.replace(out + ".tmp", out)
    return C.CDLL(out)


@pytest.mark.parametrize("factor", [1.0, 4.0, 1000.0])
def test_certain_signs_are_exact(lib, factor):
    st = adversarial_steps()
    ex = _exact_step(st)
    n = len(st)
    certain, sign = np.zeros(n, np.int32), np.zeros((n, 3), np.int32)
    args = [np.ascontiguousarray(x) for x in (st.S, st.P, st.ext, st.s, st.v, *st.a)]
    lib.probe_certain(C.c_longlong(n), *(C.c_void_p(x.ctypes.data) for x in args), C.c_float(factor),
                      C.c_void_p(certain.ctypes.data), C.c_void_p(sign.ctypes.data))
    sure = certain != 0
    assert not np.any(sure & np.any(sign != ex, axis=1))
    assert not np.any(sure & np.any(ex == 0, axis=1))
    # not vacuous where it matters, on the ordinary steps of the step's own mesh
    if factor == 1.0:
        assert sure[: len(base_steps())].mean() > 0.9
