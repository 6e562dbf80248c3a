"""The unique-edge build and the mesh extraction off the beaten track, against
the oracles: chunks of 512 tets (one below, at and past), shuffled and random
tets (more pairs in a chunk than its set holds), a vertex of thousands of edges
(a bucket past LDS), tets with a repeated vertex, far more vertices than tets
(the radix build), and an empty edge list."""
import numpy as np
import pytest

import synth
from oracle import marching_tets as MT
from oracle import regularizers as R

pytestmark = pytest.mark.gpu


def _tets(name):
    """(tets, V)"""
    rng = np.random.default_rng(7)
    grid = synth.kuhn_grid(10)[1]
    if name.startswith("grid"):
        return grid[:int(name[4:])], 11 ** 3
    if name == "shuffled":
        return grid[rng.permutation(len(grid))], 11 ** 3
    if name == "random":
        return rng.integers(0, 5000, (3000, 4)), 5000
    if name == "hub":        # vertex 3 in every tet: some 9,000 entries in its bucket
        t = rng.integers(4, 9000, (3500, 4))
        t[:, 1] = 3
        return t, 9000
    if name == "repeated":
        t = rng.integers(0, 50, (600, 4))
        t[::3, 2] = t[::3, 0]
        return t, 50
    return grid[:700] * 7, 7 * 11 ** 3 + 20000   # sparse


@pytest.mark.parametrize("name", ["grid1", "grid511", "grid512", "grid513", "grid6000", "shuffled", "random", "hub",
                                  "repeated", "sparse"])
def test_edges_bit_exact(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd.mesh import marching_tets
    from paper_2406_01579_amd.regularizers import MeshEdges
    tets, V = _tets(name)
    tets = np.ascontiguousarray(tets, np.int32)
    t = torch.as_tensor(tets, device="cuda")
    me = MeshEdges(t, V)
    assert np.array_equal(me.edges.cpu().numpy(), R.mesh_edges(tets))
    if name == "repeated":
        return   # (a flat tet's triangles are not compared)
    # the mesh: vertices in general position, so that every tet has a volume
    rng = np.random.default_rng(8)
    verts = rng.uniform(-1, 1, (V, 3)).astype(np.float32)
    sdf = rng.normal(size=V).astype(np.float32)
    keep = np.array([len(set(r)) == 4 for r in tets.tolist()])
    t = torch.as_tensor(np.ascontiguousarray(tets[keep]), device="cuda")
    pts, tris, _ = MT.extract(verts.astype(np.float64), tets[keep], sdf.astype(np.float64))
    gv, gt = marching_tets(torch.as_tensor(verts, device="cuda"), torch.as_tensor(sdf, device="cuda"), t)
    assert np.array_equal(gt.cpu().numpy(), tris)
    assert np.abs(gv.cpu().numpy() - pts).max() <= 2e-6


def test_empty_edge_list_gives_no_vertices():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd.mesh import marching_tets
    from paper_2406_01579_amd.regularizers import MeshEdges
    verts, tets = synth.kuhn_grid(4)
    v = torch.as_tensor(verts.astype(np.float32), device="cuda")
    t = torch.as_tensor(tets, device="cuda")
    me = MeshEdges(t, len(verts))
    me.count.zero_()
    gv, gt = marching_tets(v, v.norm(dim=1) - 0.7, t, me)
    assert gv.shape[0] == 0 and gt.shape[0] > 0 and bool((gt == -1).all())
