"""libqc.so is built whatever becomes of the native tensor helpers, which need torch's headers and g++."""
import ctypes
import os

import pytest

from paper_2503_06545_amd import build


@pytest.mark.parametrize("error", [FileNotFoundError("g++"), ImportError("torch")])
def test_the_library_is_linked_without_the_tensor_helpers(tmp_path, monkeypatch, capsys, error):
    objects = {s: os.path.join(build.OBJ_DIR, s.replace(".hip", ".o")) for s in build.SOURCES}
    if not all(os.path.exists(o) for o in objects.values()):
        pytest.skip("needs the objects of a build")

    def no_helpers(_=None):
        raise error

    stale = tmp_path / "_qc_torch.so"
    stale.write_bytes(b"of other sources")
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    monkeypatch.setattr(build, "RESOURCE_REPORT", str(tmp_path / "kernel_resources.txt"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libqc.so"))
    monkeypatch.setattr(build, "TORCH_LIB", str(stale))
    monkeypatch.setattr(build, "_compile", lambda s: (objects[s], [(s, "kernel", 1, 0, 1)]))
    monkeypatch.setattr(build, "_compile_roofs", lambda _=None: None)
    monkeypatch.setattr(build, "_compile_torch", no_helpers)
    assert build.build() == str(tmp_path / "libqc.so")
    assert ctypes.CDLL(str(tmp_path / "libqc.so")).qc_version() > 0
    assert not stale.exists() and "_qc_torch.so not built" in capsys.readouterr().err
