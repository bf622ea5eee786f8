"""Entry faces by projecting the boundary, with boxes far larger and far smaller
than the 64 pixels that a wavefront tests at once, shared by one or by many
wavefronts: the same faces as the tree search on every ray."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n,nu,nv,na,off", [
    (1, 257, 193, 1, 0.0),  # twelve faces, boxes of thousands of pixels, 64 wavefronts a group
    (1, 64, 64, 300, 0.0),
    (24, 31, 17, 1, 0.0),  # boxes of a pixel or none
    (8, 130, 70, 3, 0.7),  # half of the mesh beside the detector
    (20, 200, 200, 40, 0.0),
    (3, 1, 1, 5, 0.0),
])
def test_projected_entry_faces_equal_the_tree_search(n, nu, nv, na, off):
    import paper_1908_06909_amd as tct

    w = synth.jittered_kuhn(n, 81, 82, nu, nv, na)
    cone = synth.Cone(4.0, 8.0, nu, nv, 2.0 / nu, 2.0 / nv, off, -off / 2)
    mesh = tct.TetMesh(w.verts, w.tets, device=DEV)
    P = tct.Projector(mesh, tct.ConeGeometry(cone, w.angles, device=DEV), cache_entry=False)
    a, b = P.compute_entry(method="raster"), P.compute_entry(method="bvh")
    assert torch.equal(a, b)
    assert int((a >= 0).sum()) > 0
    assert np.all(a.cpu().numpy() < mesh.nboundary)
