"""The unique-edge build where a vertex is the lower end of many edges: buckets
at the ends of the three ways they are sorted (64, 2048), one with entries on
both sides of a bitmap window of 2^20 vertices, meshes of few vertices and many
tets, and tets in no order; bit for bit against the oracle.  And that none of
them costs out of proportion: a call takes at most 20 times as long as one for
as many tets of a cube grid (a sort of all pairs takes about 4 times as long)."""
import numpy as np
import pytest

import synth
from oracle import regularizers as R

pytestmark = pytest.mark.gpu


def _fan(n, rng):
    """Vertices 1, 4 and 6 are the lower ends of some n edges each (repeated over two orders of the tets)."""
    t = []
    for hub in (1, 4, 6):
        x = 10 + rng.permutation(n)
        x = np.concatenate([x, x[:-n % 3]]).reshape(-1, 3)
        t.append(np.concatenate([x[:, :1], np.full((len(x), 1), hub), x[:, 1:]], 1))
    t = np.concatenate(t)
    return np.concatenate([t, t[rng.permutation(len(t))]]), n + 10


def _mesh(name):
    rng = np.random.default_rng(3)
    kind, _, n = name.partition("-")
    n = int(n)
    if kind == "fan":
        return _fan(n, rng)
    if kind == "dense":      # 60,000 tets on n vertices
        return rng.integers(0, n, (60000, 4)), n
    if kind == "hub":        # one vertex in all of n tets
        t = rng.integers(1, n, (n, 4))
        t[:, 2] = 0
        return t, n
    if kind == "shuffled":
        v, t = synth.kuhn_grid(n)
        p = rng.permutation(len(v))
        return p[t[rng.permutation(len(t))]], len(v)
    if kind == "loose":      # more vertices than tets
        return rng.integers(0, 3 * n, (n, 4)), 3 * n
    # wide: a hub whose upper vertices lie in three windows
    V = (1 << 21) + 100
    t = rng.integers(0, V, (n, 4))
    t[:5000, 0] = 17
    t[:6, 1:] = [[17, 18, (1 << 20) + 16], [(1 << 20) + 17, (1 << 20) + 18, V - 1], [(1 << 21) + 16, (1 << 21) + 17, 48],
                 [49, 50, V - 2], [17 + (1 << 19), 17 + (1 << 20), 80], [V - 1, V - 3, V - 33]]
    return t, V


@pytest.mark.parametrize("name", ["fan-3", "fan-63", "fan-64", "fan-65", "fan-129", "fan-1023", "fan-2047", "fan-2048",
                                  "fan-2049", "fan-6000", "dense-5", "dense-300", "dense-20000", "hub-30000",
                                  "shuffled-20", "wide-2200000", "loose-3000"])
def test_edges_bit_exact(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd.regularizers import MeshEdges
    tets, V = _mesh(name)
    tets = np.ascontiguousarray(tets, np.int32)
    me = MeshEdges(torch.as_tensor(tets, device="cuda"), V)
    if len(tets) < 1000000:
        ref = R.mesh_edges(tets)
    else:   # the same in one number per pair, several times as fast
        t = tets.astype(np.int64)
        key = np.unique(np.concatenate([np.minimum(t[:, i], t[:, j]) * V + np.maximum(t[:, i], t[:, j])
                                        for i in range(4) for j in range(i + 1, 4)]))
        ref = np.stack([key // V, key % V], 1)
    assert np.array_equal(me.edges.cpu().numpy(), ref)


def _us(tets, V):
    import torch
    from paper_2406_01579_amd.regularizers import MeshEdges
    t = torch.as_tensor(np.ascontiguousarray(tets, np.int32), device="cuda")
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        MeshEdges(t, V)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("name", ["dense-60", "dense-2000", "hub-60000", "shuffled-22"])
def test_no_mesh_costs_out_of_proportion(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tets, V = _mesh(name)
    gv, gt = synth.kuhn_grid(22)
    assert _us(tets, V) <= 20.0 * _us(gt[:len(tets)], len(gv))
