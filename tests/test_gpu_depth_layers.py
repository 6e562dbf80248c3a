"""The per-tile depth sort where many entries of a list have exactly the same
depth, as the layers of a grid seen along an axis do: buckets just below, at and
past the two lengths from which a list is merge sorted, in lists that fit LDS
and longer ones, against numpy's sort by (depth bits, record)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [700, 1500, 5000])
@pytest.mark.parametrize("per", [48, 95, 96, 97, 255, 256, 257])
def test_list_order(n, per):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(n + per)
    z = (2.0 + 0.01 * rng.permutation(np.arange(n) // per)).astype(np.float32)
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
