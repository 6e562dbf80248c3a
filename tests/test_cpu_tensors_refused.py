"""Tensors that are not on the GPU are refused with ValueError before any kernel
is launched, at every entry point that takes the stream from its tensors' device."""
import types

import pytest
import torch

from paper_2406_01579_amd import Params, SceneT, _lib
from paper_2406_01579_amd import coarse, mesh, regularizers


@pytest.fixture
def launched(monkeypatch):
    """The library replaced by one that only notes which of its functions are called."""
    calls = []

    class Fake:
        def __getattr__(self, name):
            def f(*args):
                calls.append(name)
                return 0
            return f
    monkeypatch.setattr(_lib, "lib", lambda: Fake())
    return calls


def _mesh():
    v = torch.rand(5, 3)
    return v, torch.rand(5) - 0.5, torch.tensor([[0, 1, 2, 3], [1, 2, 3, 4]], dtype=torch.int32)


def _edges():
    return types.SimpleNamespace(buffer=torch.zeros(12, 2, dtype=torch.int32), count=torch.zeros(1, dtype=torch.int32),
                                 capacity=12, V=5)


def _regularizers_backward():
    v, f, t = _mesh()
    ctx = types.SimpleNamespace(saved_tensors=(v, f, t, torch.zeros(64, dtype=torch.uint8)), edges=_edges())
    regularizers.RegularizerFunction.backward(ctx, torch.ones(2, dtype=torch.float64))


CALLS = {
    "stream": lambda: _lib.current_stream(torch.device("cpu")),
    "cube_grid": lambda: coarse.cube_grid(4, torch.tensor([-1.0, -1.0, -1.0, 0.5])),
    "prefilter_bounds": lambda: coarse.prefilter_bounds(SceneT(*[_mesh()[i] for i in (0, 2, 1, 0)], 20.0), Params()),
    "refit_cube": lambda: coarse.refit_cube(torch.zeros(6), torch.zeros(4), 4),
    "coarse_to_fine": lambda: coarse.coarse_to_fine(lambda x: x[:, 0], 4, 20.0, device="cpu"),
    "marching_tets": lambda: mesh.marching_tets(*_mesh(), edges=_edges()),
    "regularizers": lambda: regularizers.regularizers(*_mesh(), _edges()),
    "regularizers_backward": _regularizers_backward,
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_refused(name, launched):
    with pytest.raises(ValueError):
        CALLS[name]()
    assert all(c.endswith("_workspace_size") for c in launched)
