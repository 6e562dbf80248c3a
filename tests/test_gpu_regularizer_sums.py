"""The block sums of the regularisers at their edges: chunks of 512 to 2048
tets (one below, at and past), a shuffled tet order whose vertices need more
groups than a block holds (the rest are added to device memory directly), and
the gradient pass on the forward's workspace, twice on one graph."""
import numpy as np
import pytest

import synth
from oracle import regularizers as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,shuffle", [(1, False), (511, False), (512, True), (513, False), (2049, True),
                                       (10368, False), (10368, True)])
def test_block_sums(K, shuffle):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd.regularizers import MeshEdges, _run, regularizers
    verts, tets = synth.kuhn_grid(12)     # 2197 vertices: 138 groups of 16
    rng = np.random.default_rng(K)
    verts = (verts + rng.uniform(-0.02, 0.02, verts.shape)).astype(np.float32)
    sdf = (np.linalg.norm(verts, axis=1) - 0.55 + rng.normal(0, 0.02, len(verts))).astype(np.float32)
    if shuffle:
        tets = tets[rng.permutation(len(tets))]
    tets = np.ascontiguousarray(tets[:K])
    w = (0.7, 1.3)
    le, ln, dv, df = R.losses_and_grads(verts.astype(np.float64), tets, sdf.astype(np.float64), *w,
                                        edges=R.mesh_edges(tets))
    t = torch.as_tensor(tets, device="cuda")
    v = torch.as_tensor(verts, device="cuda").requires_grad_(True)
    f = torch.as_tensor(sdf, device="cuda").requires_grad_(True)
    me = MeshEdges(t, len(verts))
    losses = regularizers(v, f, t, me)
    up = torch.tensor(w, dtype=torch.float64, device="cuda")
    first = torch.autograd.grad(losses, (v, f), up, retain_graph=True)
    again = torch.autograd.grad(losses, (v, f), up)
    full = torch.zeros_like(v), torch.zeros_like(f)
    l2 = _run(v.detach(), f.detach(), t, me, up.float(), *full)
    # the bars of the other regulariser tests: losses 1e-5 relative (the consistency term of one
    # tet is 0 but for rounding), gradients normwise 1e-4
    for got in (losses.detach().cpu().numpy(), l2.cpu().numpy()):
        assert abs(got[0] - le) <= 1e-5 * abs(le) + 1e-12
        assert abs(got[1] - ln) <= 1e-5 * abs(ln) + 1e-10
    for grads in (first, again, full):
        for got, ref in zip(grads, (dv, df)):
            assert np.abs(got.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max()
