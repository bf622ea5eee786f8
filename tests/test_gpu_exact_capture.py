"""One exact backprojection (mode "gather", whose scratch is allocated and given
back in the call) captured as a graph and replayed with other projections, and
eager work and synchronizations, between the replays: the bits of the eager call
each time."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_exact_backprojection_replays_the_eager_bits():
    import paper_1908_06909_amd as tct

    w = synth.jittered_kuhn(6, 95, 96, 40, 31, 5)
    mesh = tct.TetMesh(w.verts, w.tets, device=DEV)
    P = tct.Projector(mesh, tct.ConeGeometry(w.cone, w.angles, device=DEV))
    rng = np.random.default_rng(97)
    ys = [torch.as_tensor(rng.uniform(-1, 1, P.geom.nrays).astype(np.float32), device=DEV) for _ in range(4)]
    y, out = ys[0].clone(), torch.zeros(mesh.nt, device=DEV)
    P.backproject(y, mode="gather", out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.backproject(y, mode="gather", out=out)
    torch.cuda.synchronize()
    for other in ys:
        want = P.backproject(other, mode="gather")  # (eager work between the replays, with scratch of its own)
        y.copy_(other)
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        _ = P.forward(torch.rand(mesh.nt, device=DEV))
        torch.cuda.synchronize()
    assert mesh.stats(reset=True)["failed"] == 0
