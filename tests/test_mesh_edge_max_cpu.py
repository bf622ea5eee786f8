"""The longest edge of a mesh, from which the walk's step takes the bound that
its exit signs are certified under: it has to be the largest float32 coordinate
difference over all six edges of every tetrahedron, as the step forms them.  A
smaller value would certify wrong signs, a larger one would send steps to the
slower tests."""

import ctypes as C
import itertools
import os
import subprocess

import numpy as np
import pytest

import synth
from paper_1908_06909_amd import TetMesh

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1908_06909_amd", "csrc")
BUILD = os.path.join(ROOT, "_build")


def probe_lib():
    os.makedirs(BUILD, exist_ok=True)
    out, src = os.path.join(BUILD, "libmesh_probe.so"), os.path.join(HERE, "mesh_probe.cpp")
    if not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(f) for f in
                                                              (src, os.path.join(CSRC, "common.h"))):
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "-O2",
                        "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc", "-Wno-unused-command-line-argument", "-I",
                        CSRC, "-I", os.path.join(ROOT, "include"), src, "-o", out + ".tmp"],
                       check=True, capture_output=True)
        os.replace(out + ".tmp", out)
    return C.CDLL(out)


@pytest.fixture(scope="module")
def edge_max():
    fn = probe_lib().probe_edge_max
    fn.argtypes, fn.restype = [C.c_void_p], C.c_float
    return fn


def _want(verts, tets):
    p = np.asarray(verts, np.float32)[np.asarray(tets)]
    return max(float(np.abs(p[:, i] - p[:, j]).max()) for i, j in itertools.combinations(range(4), 2))


def _meshes():
    w = synth.jittered_kuhn(6, 91, 92, 8, 8, 1)
    yield "jittered", w.verts, w.tets
    yield ("delaunay", *synth.delaunay_mesh(2000, 5))
    X = synth.graded_nodes(12, 1.3, 5)
    yield ("graded", *synth.kuhn_mesh(X, X, synth.kuhn_nodes(4)))


@pytest.mark.parametrize("name,verts,tets", list(_meshes()))
def test_longest_edge_of_a_mesh(edge_max, name, verts, tets):
    for reorder in (True, False):
        m = TetMesh(verts, tets, host_only=True, reorder=reorder)
        assert edge_max(m.handle) == _want(verts, tets)


@pytest.mark.parametrize("pair", list(itertools.combinations(range(4), 2)))
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_each_edge_and_axis_counts(edge_max, pair, axis):
    """One tetrahedron whose longest difference lies along one edge and axis,
    with coordinates whose difference is rounded."""
    verts = np.array([[0.1, 0.2, 0.3], [0.4, 0.2, 0.1], [0.2, 0.5, 0.2], [0.3, 0.3, 0.6]], np.float32)
    verts[pair[0], axis], verts[pair[1], axis] = -7.3, 7.1000001
    want = float(np.abs(verts[pair[0], axis] - verts[pair[1], axis]))
    assert want == _want(verts, [[0, 1, 2, 3]])
    assert edge_max(TetMesh(verts, [[0, 1, 2, 3]], host_only=True).handle) == want
