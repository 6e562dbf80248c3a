"""The multi-wave 8x8 kernels evaluate only the pixels inside a record's hull
spans; the one-wave kernel evaluates its whole rectangle.  Images of the two
are equal bit for bit, so a span that left out a covered pixel would show: on
soups of random tets from under a pixel to the whole image (spans in units of
1 to 64 pixels), flattened ones (thin faces) and cameras inside the soup
(tets across the near plane, coordinates of millions of pixels)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _soup(n, seed, lo, hi, flat):
    rng = np.random.default_rng(seed)
    size = np.exp(rng.uniform(np.log(lo), np.log(hi), size=(n, 1, 1)))
    x = rng.normal(size=(n, 4, 3)) * size
    if flat:   # squash every tet along a direction of its own
        d = rng.normal(size=(n, 1, 3))
        d /= np.linalg.norm(d, axis=2, keepdims=True)
        x -= (1.0 - 10.0 ** rng.uniform(-6, 0, size=(n, 1, 1))) * (x * d).sum(2, keepdims=True) * d
    x += rng.uniform(-1, 1, size=(n, 1, 3))
    sdf = rng.normal(0.0, 0.05, size=4 * n)
    return synth.Scene(x.reshape(-1, 3).astype(np.float32), np.arange(4 * n, dtype=np.int32).reshape(n, 4),
                       sdf.astype(np.float32), rng.uniform(size=(4 * n, 3)).astype(np.float32), 20.0)


@pytest.mark.parametrize("lo,hi,flat,radius,W,H", [
    (0.003, 0.03, False, 2.5, 333, 217),
    (0.01, 0.3, False, 2.5, 1024, 640),
    (0.02, 1.0, True, 2.5, 517, 389),
    (0.01, 0.5, True, 0.3, 200, 331),
    (0.05, 0.8, False, 0.3, 64, 48),
])
def test_spans_leave_out_no_covered_pixel(lo, hi, flat, radius, W, H):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    sc = SceneT.from_numpy(_soup(4000, 11, lo, hi, flat))
    cams = np.stack([synth.orbit_camera(az, 0.3, radius, 50.0, W, H, znear=1e-3) for az in (0.4, 2.9)])
    for params in (Params.exact, Params):   # without thresholds every covered pixel counts
        a = Renderer(params(waves=4)).forward([sc], cams)
        b = Renderer(params(waves=1)).forward([sc], cams)
        for x, y in zip(a.outs, b.outs):
            assert torch.equal(x.nan_to_num(), y.nan_to_num())
