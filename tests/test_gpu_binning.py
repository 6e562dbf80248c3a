"""Binning at its edges, bit for bit against the oracle's brute-force lists:
records over thousands of tiles (more tiles in a round than the hash of tiles
holds, several rounds per block), more than 64 blocks of tiles (their counts
summed by a launch of their own), a single tile; and a forward whose entries
exceed the capacity leaves every list empty."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import gpu_forward, gpu_tiling, oracle_params

pytestmark = pytest.mark.gpu


def _soup(n, lo, hi):
    rng = np.random.default_rng(n)
    size = np.exp(rng.uniform(np.log(lo), np.log(hi), size=(n, 1, 1)))
    x = rng.normal(size=(n, 4, 3)) * size + rng.uniform(-1, 1, size=(n, 1, 3))
    return synth.Scene(x.reshape(-1, 3).astype(np.float32), np.arange(4 * n, dtype=np.int32).reshape(n, 4),
                       rng.normal(0.0, 0.05, size=4 * n).astype(np.float32),
                       rng.uniform(size=(4 * n, 3)).astype(np.float32), 20.0)


@pytest.mark.parametrize("n,lo,hi,W,H,tile", [(300, 0.3, 1.5, 700, 500, (8, 8)), (300, 0.3, 1.5, 333, 217, (16, 8)),
                                              (900, 0.01, 0.3, 2100, 2100, (8, 8)), (700, 0.01, 0.3, 8, 8, (8, 8))])
def test_lists_bit_exact(n, lo, hi, W, H, tile):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params
    sc = _soup(n, lo, hi)
    cams = np.stack([synth.orbit_camera(az, 0.3, 2.5, 50.0, W, H) for az in (0.4, 2.9)])
    P = Params(tile_w=tile[0], tile_h=tile[1])
    r, plan, _ = gpu_forward(sc, cams, P)
    d, tets = gpu_tiling(r, plan)
    ref = oracle.binning(oracle.Geometry.of(sc), cams, oracle_params(P, 20.0))
    assert d["entries"] == ref["E"]
    assert np.array_equal(d["tile_keys"], ref["tile"].astype(np.uint32))
    assert np.array_equal(tets, ref["tet"])
    assert np.array_equal(d["ranges"].astype(np.int64), ref["ranges"].astype(np.int64))


def test_overflow_leaves_empty_lists():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_01579_amd import Params, Renderer, SceneT
    sc = SceneT.from_numpy(_soup(300, 0.1, 0.5))
    cams = synth.orbit_camera(0.4, 0.3, 2.5, 50.0, 200, 120, bg=(0.25, 0.5, 0.75))[None]
    r = Renderer(Params(), check="none")
    plan = r.forward([sc], cams, caps=(300, 64))
    s = r.read_status(plan)
    assert s.overflow == 2 and s.entries == 64 and s.entries_needed > 64
    assert not r.debug(plan)["ranges"].any()
    grads, = r.backward(plan, [torch.ones((8, 120, 200), device="cuda")])
    assert not any(bool(g.any()) for g in grads)
    bg = torch.tensor([0.25, 0.5, 0.75, 0, 0, 0, 0, 0], device="cuda")[:, None, None]
    assert torch.equal(plan.outs[0], bg.expand(8, 120, 200))
