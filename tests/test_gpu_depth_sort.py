"""The per-tile depth sort at its edges: lists of one to several thousand
entries in one tile (one LDS load, groups of buckets), depths spread evenly,
in two tight clusters, a few ulps apart and all equal (crowded buckets: the
merge sort), against numpy's sort by (depth bits, record), which is exact: the
camera's depth is the vertices' z."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _depths(kind, n, rng):
    if kind == "spread":
        return rng.uniform(1.0, 4.0, n).astype(np.float32)
    if kind == "clusters":   # nearly all in two narrow bands of a wide range
        z = np.where(rng.uniform(size=n) < 0.5, 1.5, 3.0) + rng.normal(0.0, 1e-5, n)
        z[:1], z[-1:] = 1.0, 4.0
        return z.astype(np.float32)
    if kind == "ulps":
        return (np.float32(2.0) + rng.integers(0, 8, n).astype(np.float32) * np.float32(2.0 ** -22)).astype(np.float32)
    return np.full(n, 2.0, np.float32)


@pytest.mark.parametrize("kind", ["spread", "clusters", "ulps", "equal"])
@pytest.mark.parametrize("n", [1, 2, 49, 256, 257, 1024, 1025, 2048, 2049, 5000])
def test_list_order(kind, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(n)
    z = _depths(kind, n, rng)
    corner = np.array([[-0.2, -0.2], [0.2, -0.2], [0.0, 0.2], [0.05, 0.0]], np.float32)
    x = np.empty((n, 4, 3), np.float32)
    x[:, :, :2] = corner * z[:, None, None]       # all inside the one tile
    x[:, :, 2] = z[:, None]
    sdf = np.tile(np.array([0.1, 0.1, 0.1, -0.1], np.float32), n)
    sc = SceneT.from_numpy(synth.Scene(x.reshape(-1, 3), np.arange(4 * n, dtype=np.int32).reshape(n, 4), sdf,
                                       np.ones((4 * n, 3), np.float32), 20.0))
    cam = np.zeros((1, 22), np.float32)
    cam[0, :2] = 8, 8
    cam[0, 2:11] = np.eye(3, dtype=np.float32).ravel()
    cam[0, 14:19] = 8.0, 8.0, 4.0, 4.0, 0.01
    r = Renderer(Params())
    d = r.debug(r.forward([sc], cam))
    assert d["entries"] == n
    zt = ((x[:, 0, 2] + x[:, 1, 2]) + (x[:, 2, 2] + x[:, 3, 2])) * np.float32(0.25)
    assert np.array_equal(d["entry_record"], np.lexsort((np.arange(n), zt)))
    assert not d["tile_keys"].any()
