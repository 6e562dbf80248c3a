"""The pair-gradient kernel at the edges of its windows (448 pairs, segments of
1 to 64 pairs that end before, at and past a window's end): gradients of the
multi-wave path against the one-wave kernel, which chains and sums each
(entry, pixel) on its own, normwise to the 1e-4 bar of the other gradient
tests; and the deterministic mode repeats bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lo,hi,W,H", [(1, 1.0, 1.0, 8, 8), (7, 1.2, 1.2, 8, 8), (8, 1.5, 1.5, 16, 8),
                                         (40, 0.3, 0.8, 64, 48), (500, 0.02, 0.3, 200, 120),
                                         (3000, 0.01, 0.05, 333, 217)])
def test_pair_windows(n, lo, hi, W, H):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(n)
    size = np.exp(rng.uniform(np.log(lo), np.log(hi), size=(n, 1, 1)))
    corner = np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]], float)
    x = (corner + 0.3 * rng.normal(size=(n, 4, 3))) * size + (rng.uniform(-1, 1, size=(n, 1, 3)) if n > 8 else 0.0)
    # f falls away from the camera (a tet whose f rises along the ray is transparent)
    to_cam = np.array([np.cos(0.3) * np.cos(0.4), np.cos(0.3) * np.sin(0.4), np.sin(0.3)])
    f = 0.1 * x.reshape(-1, 3) @ to_cam + rng.normal(0.0, 0.02, size=4 * n)
    sc = SceneT.from_numpy(synth.Scene(x.reshape(-1, 3).astype(np.float32),
                                       np.arange(4 * n, dtype=np.int32).reshape(n, 4), f.astype(np.float32),
                                       rng.uniform(size=(4 * n, 3)).astype(np.float32), 20.0))
    cams = synth.orbit_camera(0.4, 0.3, 2.5, 50.0, W, H)[None]
    douts = [torch.as_tensor(rng.normal(size=(8, H, W)).astype(np.float32), device="cuda")]

    def grads(**kw):
        r = Renderer(Params(**kw))
        return r.backward(r.forward([sc], cams), douts)[0]
    ref = grads(waves=1)
    got = grads(waves=4)
    det = grads(waves=4, deterministic=True)
    for g, d, d2, w in zip(got, det, grads(waves=4, deterministic=True), ref):
        top = float(w.abs().max())
        assert top > 0.0
        assert float((g - w).abs().max()) <= 1e-4 * top
        assert float((d - w).abs().max()) <= 1e-4 * top
        assert torch.equal(d, d2)
