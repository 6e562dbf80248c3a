"""The lists that the multi-wave kernels walk leave out the entries that cannot
blend (their tet faces away from the camera, or covers no pixel centre); the
one-wave kernel walks the full lists.  Both give the same images bit for bit,
the same last blended entry (an index into the full list) and gradients to the
1e-4 bar of the other gradient tests: with f falling away from the camera
(nothing left out but slivers), rising (whole lists left out), both, and random;
at steepnesses where the rule may leave out much and nothing; and without
thresholds, where a transparent tet counts as blended."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _scene(kind, n, s, rng):
    verts, tets = synth.kuhn_grid(n)
    to_cam = np.array([np.cos(0.3) * np.cos(0.4), np.cos(0.3) * np.sin(0.4), np.sin(0.3)])
    x = verts @ to_cam
    f = {"falls": x, "rises": -x, "both": np.abs(x) - 0.5, "noise": rng.normal(size=len(verts))}[kind]
    return synth.Scene(verts.astype(np.float32), tets, (f * 6.0 / s + rng.normal(0.0, 0.02 / s, len(verts))).astype(np.float32),
                       rng.uniform(size=(len(verts), 3)).astype(np.float32), s)


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("s", [20.0, 320.0, 1e5])
@pytest.mark.parametrize("kind,n,W,H", [("falls", 9, 100, 75), ("rises", 9, 100, 75), ("both", 16, 333, 217),
                                        ("noise", 6, 64, 64)])
def test_same_as_the_full_lists(kind, n, W, H, s, exact):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    rng = np.random.default_rng(n)
    sc = SceneT.from_numpy(_scene(kind, n, s, rng))
    cams = np.stack([synth.orbit_camera(az, 0.3, 2.5, 50.0, W, H) for az in (0.4, 2.9)])
    douts = [torch.as_tensor(rng.normal(size=(8, H, W)).astype(np.float32), device="cuda") for _ in cams]
    make = Params.exact if exact else Params
    res = []
    for waves in (1, 4):
        r = Renderer(make(waves=waves))
        plan = r.forward([sc], cams)
        res.append((plan.outs, r.debug(plan), r.backward(plan, douts)[0]))
    (oa, da, ga), (ob, db, gb) = res
    for a, b in zip(oa, ob):
        assert torch.equal(a, b)
    assert np.array_equal(da["entry_record"], db["entry_record"])
    assert np.array_equal(da["last"], db["last"]) and np.array_equal(da["t_last"], db["t_last"])
    for a, b in zip(ga, gb):
        assert float((a - b).abs().max()) <= 1e-4 * max(float(a.abs().max()), 1e-30)
