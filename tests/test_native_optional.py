"""Without _gridtorch.so (no torch headers where the library was built) the torch-facing calls
keep to ctypes: nothing raises because the module is missing."""
import os

import pytest

from paper_2109_06976_amd import build, grid


@pytest.fixture
def no_module(monkeypatch, tmp_path):
    monkeypatch.setattr(grid, "_NATIVE_PATH", str(tmp_path / "_gridtorch.so"))
    monkeypatch.setattr(grid, "_native_mod", None)


class Model:
    """What the wrappers read of a model that is closed: the library refuses its handle."""
    n, device, _h, handle = 7, 0, None, None
    fd = grid.Model.fd


def test_calls_take_ctypes_without_the_native_module(no_module):
    import torch
    x = torch.zeros((2, 7))
    assert grid._plain_torch(x)
    assert grid._native() is None
    assert not grid._launch("grid_fd", Model, 2, (x, x, x, x), (14,) * 4, None)
    with pytest.raises(grid.GridError) as e:       # the binding's own check of a buffer
        Model().fd(x, x, x, x)
    assert e.value.status == grid.GRID_EINVAL and "not a GPU tensor" in str(e.value)


def test_build_leaves_the_native_module_out_without_torch_headers(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "torch_root", lambda: None)
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    assert build.build_torch_module() is None
    assert os.listdir(tmp_path) == []
