"""The scatters' wavefront tables where they are fullest and smallest: rays so
far apart that a window meets more tetrahedra than the table has slots (probes
wrap around, terms go straight to memory, windows are halved), meshes whose
tetrahedra do not fill the table's groups of four, and a detector of odd size.
Every element against the oracle, within the bars of the other backprojection
tests."""

import numpy as np
import pytest
import torch

import oracle
import synth
from parity_bars import assert_within, backprojection_reference, element_size

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SHAPES = {
    "crowded": (24, 40, 24, 8),  # 64 rays, few tetrahedra in common
    "one cell": (1, 33, 17, 5),  # six tetrahedra
    "part of a group": (3, 48, 48, 7),  # 162 tetrahedra
}


@pytest.mark.parametrize("mode", ["atomic", "fixed", "gather"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_scatter_tables_at_their_edges(shape, mode):
    import paper_1908_06909_amd as tct

    n, nu, nv, na = SHAPES[shape]
    w = synth.jittered_kuhn(n, 51, 52, nu, nv, na)
    orc = oracle.Oracle(w.verts, w.tets, w.cone, w.angles)
    mesh = tct.TetMesh(w.verts, w.tets, device=DEV)
    P = tct.Projector(mesh, tct.ConeGeometry(w.cone, w.angles, device=DEV))
    H = element_size(w.verts, w.tets, orc.mesh.tables()[1])
    y = np.random.default_rng(53).uniform(-1, 1, orc.nrays).astype(np.float32)
    ref, tol = backprojection_reference(orc, y, H, float_atomic=mode == "atomic")
    got = mesh.to_user(P.backproject(torch.as_tensor(y, device=DEV), mode=mode)).cpu().numpy()
    assert_within(got, ref, tol, f"{shape} {mode}")
    assert mesh.stats(reset=True)["failed"] == 0
