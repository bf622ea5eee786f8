"""The exact backprojection (mode "gather") where its accumulators work
hardest: projections whose rays are up to 2^100 apart in strength, so that a
tetrahedron's partial sums fall into different words and weak ones must not be
lost beside strong ones elsewhere.  Every element against the oracle, at bars
relative to the rays that cross that element; the same bits on every run, and
for an angle range added to the rest."""

import numpy as np
import pytest
import torch

import oracle
import synth
from parity_bars import assert_within, backprojection_reference, element_size

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("spread", [0, 60, 100])
@pytest.mark.parametrize("na", [1, 6])
def test_weak_rays_keep_their_precision(spread, na):
    import paper_1908_06909_amd as tct

    w = synth.jittered_kuhn(6, 61, 62, 70, 52, na)
    orc = oracle.Oracle(w.verts, w.tets, w.cone, w.angles)
    mesh = tct.TetMesh(w.verts, w.tets, device=DEV)
    P = tct.Projector(mesh, tct.ConeGeometry(w.cone, w.angles, device=DEV))
    H = element_size(w.verts, w.tets, orc.mesh.tables()[1])
    rng = np.random.default_rng(63)
    # Strength grows along the columns and falls along the rows.
    level = np.linspace(-0.5, 0.5, 70)[None, :] - 0.3 * np.linspace(-0.5, 0.5, 52)[:, None]
    y = (rng.uniform(-1, 1, (na, 52, 70)) * 2.0 ** (spread * level)).astype(np.float32)
    ref, tol = backprojection_reference(orc, y.ravel(), H)
    yt = torch.as_tensor(y, device=DEV)
    a = P.backproject(yt, mode="gather")
    assert torch.equal(a, P.backproject(yt, mode="gather"))
    assert_within(mesh.to_user(a).cpu().numpy(), ref, tol, f"spread 2^{spread}, {na} angles")
    if na > 1:
        part = P.backproject_range(yt, 0, 2, mode="gather")
        both = P.backproject_range(yt, 2, na - 2, mode="gather", out=part, accumulate=True)
        assert_within(mesh.to_user(both).cpu().numpy(), ref, 2 * tol, f"spread 2^{spread}, two ranges")
    assert mesh.stats(reset=True)["failed"] == 0
