"""Marching tetrahedra on a part of a mesh with the edge list of the whole: edges
with an end past the part's vertices lie among its own and are left out, whichever
lanes they fall on."""
import numpy as np
import pytest

import synth
from oracle import marching_tets as MT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,V", [(6, 100), (12, 700), (12, 2000)])
def test_edges_of_a_larger_mesh(R, V):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd.mesh import marching_tets
    from paper_2406_01579_amd.regularizers import MeshEdges
    verts, tets = synth.kuhn_grid(R)
    rng = np.random.default_rng(R)
    p = rng.permutation(len(verts))       # the part's vertices are all over the mesh
    tets = np.ascontiguousarray(p[tets], np.int32)
    x = np.empty_like(verts)
    x[p] = verts
    own = tets[(tets < V).all(1)]
    sdf = rng.normal(size=V).astype(np.float32)
    pts, tris, _ = MT.extract(x[:V].astype(np.float64), own, sdf.astype(np.float64))
    # the whole list numbers the part's surface vertices by its own crossed edges
    whole = MeshEdges(torch.as_tensor(tets, device="cuda"), len(verts))
    e = whole.edges.cpu().numpy()
    e = e[(e < V).all(1)]
    cut = e[(sdf[e[:, 0]] < 0) != (sdf[e[:, 1]] < 0)]
    gv, gt = marching_tets(torch.as_tensor(x[:V].astype(np.float32), device="cuda"), torch.as_tensor(sdf, device="cuda"),
                           torch.as_tensor(own, device="cuda"), whole)
    assert gv.shape[0] == len(cut) and gt.shape[0] == len(tris) > 0
    gv, gt = gv.cpu().numpy(), gt.cpu().numpy()
    assert np.abs(gv[gt] - pts[tris]).max() <= 2e-6
