"""The kernels of the build are compiled by the compiler that built the library, also when the
building process has imported torch (whose own hiprtc is of another release)."""
import os

from paper_2109_06976_amd import build


def objects(folder):
    return {f: open(os.path.join(folder, f), "rb").read() for f in os.listdir(folder)
            if f.endswith(".hsaco")}


def test_kernels_come_from_the_hip_compiler(tmp_path, monkeypatch):
    import torch  # noqa: F401
    (tmp_path / "grid_0.hsaco").write_bytes(b"made by some other compiler")
    monkeypatch.setenv("GRID_KERNEL_CACHE", str(tmp_path))
    mark = build.compiler_id()
    assert b"clang version" in mark
    build.precompile(names=[build.tree_models()["pairs8"].name])
    made = objects(tmp_path)
    assert len(made) == 2 and "grid_0.hsaco" not in made
    for name, data in made.items():
        assert mark in data, name
