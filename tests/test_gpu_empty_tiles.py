"""Mostly empty images: fewer entries than tiles, with the entry capacity at
exactly what the call needs (launches are bounded by it), one tet per tile and
one small object, and no entry at all; the multi-wave and the resort-window
kernels against the one-wave kernel and against ample capacities, and the tile
counters of an image of many tiles, which few blocks of tets clear; and an image
of more lists than the depth sort launches workgroups."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _specks(n, W):
    """n tets of under a pixel, each in a tile of its own."""
    rng = np.random.default_rng(n)
    tiles = rng.choice((W // 8) ** 2, n, replace=False)
    px = (np.stack([tiles % (W // 8), tiles // (W // 8)], 1) * 8 + 4.5) / W - 0.5   # a pixel's centre
    corner = np.array([[-0.6, -0.5], [0.7, -0.4], [0.0, 0.7], [0.1, 0.0]]) / W
    x = np.empty((n, 4, 3), np.float32)
    x[:, :, :2] = (px[:, None] + corner) * 2.0
    x[:, :, 2] = 2.0 + np.array([0.0, 0.0, 0.0, -0.01])
    sdf = np.tile(np.array([-0.1, -0.1, -0.1, 0.1], np.float32), n)
    return synth.Scene(x.reshape(-1, 3), np.arange(4 * n, dtype=np.int32).reshape(n, 4), sdf,
                       rng.uniform(size=(4 * n, 3)).astype(np.float32), 20.0)


def _small(W):
    verts, tets = synth.kuhn_grid(6)
    rng = np.random.default_rng(W)
    x = verts * 0.05 + np.array([0.3, -0.2, 2.0])
    sdf = np.linalg.norm(verts, axis=1) - 0.7 + rng.normal(0.0, 0.01, len(verts))
    return synth.Scene(x.astype(np.float32), tets, sdf.astype(np.float32), rng.uniform(size=(len(verts), 3)).astype(np.float32), 20.0)


@pytest.mark.parametrize("kind,W", [("specks", 512), ("small", 512), ("small", 2048), ("none", 512)])
@pytest.mark.parametrize("kw", [dict(), dict(recompute_state=True), dict(window=3), dict(waves=2, chunk_bwd=16)])
def test_capacity_below_the_tiles(kind, W, kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    sc = _specks(700, W) if kind == "specks" else _small(W)
    if kind == "none":
        sc.verts[:, 2] -= 10.0
    sc = SceneT.from_numpy(sc)
    cam = np.zeros((1, 22), np.float32)
    cam[0, :2] = W, W
    cam[0, 2:11] = np.eye(3, dtype=np.float32).ravel()
    cam[0, 14:19] = W, W, W / 2, W / 2, 0.01
    cam[0, 19:22] = 0.2, 0.4, 0.6
    dout = [torch.as_tensor(np.random.default_rng(1).normal(size=(8, W, W)).astype(np.float32), device="cuda")]
    params = Params.exact(**kw)
    ample = Renderer(params)
    plan = ample.forward([sc], cam, caps=(0, 1 << 20))
    st = ample.read_status(plan)
    assert st.entries < (W // 8) ** 2 and st.overflow == 0
    assert (st.entries == 0) == (kind == "none")
    ref, gref = plan.outs[0], ample.backward(plan, dout)[0]
    tight = Renderer(params, check="none")
    plan = tight.forward([sc], cam, caps=(0, max(1, int(st.entries_needed))))
    assert tight.read_status(plan).overflow == 0
    assert torch.equal(plan.outs[0], ref)
    got = tight.backward(plan, dout)[0]
    one = Renderer(Params.exact(waves=1)).forward([sc], cam)
    if not kw.get("window"):
        assert torch.equal(one.outs[0], ref)
    for a, b in zip(got, gref):
        assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max())
    if kind != "none":
        assert float(gref[1].abs().max()) > 0.0


def test_more_lists_than_sort_workgroups():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    W = 2048   # 65536 tiles, every one inside the projection of a cube's six tets
    verts, tets = synth.kuhn_grid(1)
    rng = np.random.default_rng(2)
    verts = verts * np.array([40.0, 40.0, 1.0]) + np.array([0.0, 0.0, 3.0]) + rng.normal(0.0, 0.1, verts.shape)
    sc = synth.Scene(verts.astype(np.float32), tets, rng.normal(0.0, 0.1, len(verts)).astype(np.float32),
                     rng.uniform(size=(len(verts), 3)).astype(np.float32), 20.0)
    cam = np.zeros((1, 22), np.float32)
    cam[0, :2] = W, W
    cam[0, 2:11] = np.eye(3, dtype=np.float32).ravel()
    cam[0, 14:19] = W, W, W / 2, W / 2, 0.01
    r = Renderer(Params(prefilter_tf=0.0))
    d = r.debug(r.forward([SceneT.from_numpy(sc)], cam))
    lens = d["ranges"][:, 1] - d["ranges"][:, 0]
    assert (lens >= 2).sum() > 32768
    z = sc.verts[:, 2][sc.tets[d["kept_tet"]]]
    zt = ((z[:, 0] + z[:, 1]) + (z[:, 2] + z[:, 3])) * np.float32(0.25)
    rec, tile = d["entry_record"], d["tile_keys"]
    assert np.array_equal(tile, np.repeat(np.arange(len(lens)), lens))
    assert np.array_equal(np.lexsort((rec, zt[rec], tile)), np.arange(len(rec)))
