"""Loading the package without a _marshal.so that fits this PyTorch: a warning, and every call through ctypes."""
import os

import pytest

import paper_2410_03355_amd as lantern
from paper_2410_03355_amd import binding


@pytest.mark.parametrize("kind", ["missing", "no library", "other version"])
def test_library_loads_without_its_host_half(monkeypatch, tmp_path, kind):
    if not os.path.exists(lantern.LIB_PATH):
        lantern.build()
    if kind == "other version":
        monkeypatch.setattr(binding, "marshal_built_for", lambda: "PyTorch 0.0, Python 3.0", raising=False)
    else:
        path = tmp_path / "_marshal.so"
        monkeypatch.setattr(binding, "MARSHAL_PATH", str(path))
        if kind == "no library":
            path.write_bytes(b"not a library")
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_marshal", None)
    with pytest.warns(RuntimeWarning, match="_marshal.so"):
        lib = binding.load()
    assert lib.lantern_version() > 0
    for call in ("verify", "decide_rows", "verify_trees_sequential", "accept_chains"):
        assert getattr(binding._marshal, call)(None) is None      # declined: the way through ctypes
