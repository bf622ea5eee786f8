"""The element-driven backprojection at the shapes its loops can get wrong:
shadows of thousands of pixels (few elements: chunks of angles, and an exact
pass whose lanes take pixels), shadows smaller than a pixel, one-pixel-wide
detectors, and rays through nodes and along edges in each (an unjittered mesh
and symmetric detectors), so that elements do reach the exact pass.  Every
element against the oracle, and the same bits twice."""

import numpy as np
import pytest
import torch

import oracle
import synth
from parity_bars import assert_within, backprojection_reference, element_size

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SHAPES = {
    "large shadows, ties": ("plain", 2, 95, 79, 6),
    "large shadows, many angles": ("plain", 2, 40, 33, 70),
    "small shadows": ("jittered", 14, 9, 7, 5),
    "small shadows, ties": ("plain", 12, 13, 11, 4),
    "one column": ("plain", 4, 1, 65, 6),
    "one row": ("jittered", 4, 65, 1, 20),
    "more columns than the table in LDS holds": ("jittered", 3, 2300, 3, 3),
}


@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_shadow_backprojection_shapes(shape):
    import paper_1908_06909_amd as tct

    kind, n, nu, nv, na = SHAPES[shape]
    w = synth.jittered_kuhn(n, 71, 72, nu, nv, na) if kind == "jittered" else synth.plain_kuhn(n, 72, nu, nv, na)
    w.cone = synth.Cone(4.0, 8.0, nu, nv, 2.0 / nu, 2.0 / nv)
    orc = oracle.Oracle(w.verts, w.tets, w.cone, w.angles)
    mesh = tct.TetMesh(w.verts, w.tets, device=DEV)
    P = tct.Projector(mesh, tct.ConeGeometry(w.cone, w.angles, device=DEV))
    H = element_size(w.verts, w.tets, orc.mesh.tables()[1])
    y = np.random.default_rng(73).uniform(-1, 1, orc.nrays).astype(np.float32)
    ref, tol = backprojection_reference(orc, y, H)
    yt = torch.as_tensor(y, device=DEV)
    mesh.stats(reset=True)
    a = P.backproject(yt, mode="shadow")
    exact = mesh.stats(reset=True)["exact_stage"]
    assert torch.equal(a, P.backproject(yt, mode="shadow"))
    assert_within(mesh.to_user(a).cpu().numpy(), ref, tol, shape)
    assert exact > 0 or kind == "jittered"
