"""Pixels that are NaN in one image and a number in the other would be equal after
nan_to_num: where NaN colours, positions and SDF values make NaN pixels, the
multi-wave kernels (hull spans, blend lists) have them at the same pixels as the
one-wave kernel, which evaluates every record's whole rectangle, and equal numbers
elsewhere."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["colors", "verts", "sdf", "inf"])
@pytest.mark.parametrize("radius", [2.5, 0.3])
def test_same_nan_pixels(what, radius):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(17)
    n = 1500
    x = rng.normal(size=(n, 4, 3)) * np.exp(rng.uniform(np.log(0.01), np.log(0.4), (n, 1, 1))) + rng.uniform(-1, 1, (n, 1, 3))
    x = x.reshape(-1, 3).astype(np.float32)
    sdf = rng.normal(0.0, 0.05, 4 * n).astype(np.float32)
    colors = rng.uniform(size=(4 * n, 3)).astype(np.float32)
    bad = rng.choice(4 * n, 12, replace=False)
    {"colors": colors, "verts": x, "sdf": sdf[:, None], "inf": x}[what][bad] = np.inf if what == "inf" else np.nan
    sc = SceneT.from_numpy(synth.Scene(x, np.arange(4 * n, dtype=np.int32).reshape(n, 4), sdf, colors, 20.0))
    cams = np.stack([synth.orbit_camera(az, 0.3, radius, 50.0, 200, 331, znear=1e-3) for az in (0.4, 2.9)])
    for params in (Params.exact, Params):
        outs = [Renderer(params(waves=w)).forward([sc], cams).outs for w in (4, 1)]
        for a, b in zip(*outs):
            assert torch.equal(a.isnan(), b.isnan())
            assert torch.equal(a.nan_to_num(), b.nan_to_num())
            if what == "colors" and radius > 1.0:   # (a camera in the soup may see none of the few)
                assert bool(a.isnan().any()) and not bool(a[3].isnan().any())
