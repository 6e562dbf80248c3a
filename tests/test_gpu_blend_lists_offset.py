"""Inside an object the SDF is far from zero and may be almost flat; a pair's two
interpolated values are then rounded to more than they differ by, and at a high
steepness that alone can blend.  The multi-wave kernels, whose lists leave out
the tets that cannot blend, agree with the one-wave kernel there bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset,span,s", [(-0.1, 5e-8, 1e6), (-0.1, 1e-5, 1e5), (-3.0, 1e-6, 3e4), (-100.0, 1e-4, 320.0)])
def test_same_as_the_full_lists(offset, span, s):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(5)
    verts, tets = synth.kuhn_grid(9)
    away = -(verts @ np.array([np.cos(0.3) * np.cos(0.4), np.cos(0.3) * np.sin(0.4), np.sin(0.3)]))
    sdf = offset + span * (away + 0.05 * rng.normal(size=len(verts)))
    sc = SceneT.from_numpy(synth.Scene(verts.astype(np.float32), tets, sdf.astype(np.float32),
                                       rng.uniform(size=(len(verts), 3)).astype(np.float32), s))
    cams = np.stack([synth.orbit_camera(az, 0.3, 2.5, 50.0, 333, 217) for az in (0.4, 2.9)])
    outs = [Renderer(Params(waves=w)).forward([sc], cams).outs for w in (1, 4)]
    for a, b in zip(*outs):
        assert torch.equal(a, b)
