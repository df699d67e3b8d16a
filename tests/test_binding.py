"""The Python binding's per-step calls on both of their routes, the C argument converter (csrc/pycall.cpp) and ctypes,
and the converter's build (no GPU: every call here fails at its checks or at the first HIP call, so the module is
skipped where a GPU is visible)."""
import importlib.machinery
import os
import warnings

import pytest
import torch

from paper_2606_01483_amd import _build
from paper_2606_01483_amd import murmur as M

pytestmark = pytest.mark.skipif(torch.cuda.device_count() > 0, reason="host-only checks run where no GPU is visible")


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(M.LIB_PATH):
        _build.build()
    M.lib()


# ---- the converter's build ---------------------------------------------------------------------------------------

def fake_build(monkeypatch, tmp_path, fail):
    """_build.build() into tmp_path with its commands replaced: each creates its output, the converter's fails."""
    def run(cmd):
        if fail and any(str(c).endswith("pycall.cpp") for c in cmd):
            raise RuntimeError("build step failed (1): Python.h: No such file or directory")
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("built")
    monkeypatch.setattr(_build, "_run", run)
    monkeypatch.setattr(_build, "PKG", str(tmp_path))
    monkeypatch.setattr(_build, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(_build, "LIB", str(tmp_path / "libmurmur.so"))
    monkeypatch.setattr(_build, "PYCALL", str(tmp_path / os.path.basename(_build.PYCALL)))


def test_build_without_the_converter(monkeypatch, tmp_path):
    """Where the converter does not compile (no Python headers) the library is built all the same, and no converter
    of an earlier build stays beside it, whose calls might be laid out for another library."""
    fake_build(monkeypatch, tmp_path, fail=True)
    (tmp_path / os.path.basename(_build.PYCALL)).write_text("old")
    (tmp_path / "_pycall.so").write_text("older")
    with pytest.warns(UserWarning, match="Python.h"):
        assert _build.build() == str(tmp_path / "libmurmur.so")
    assert (tmp_path / "libmurmur.so").read_text() == "built"
    assert [f for f in os.listdir(tmp_path) if "pycall" in f] == []
    fake_build(monkeypatch, tmp_path, fail=False)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        _build.build()
    assert (tmp_path / os.path.basename(_build.PYCALL)).read_text() == "built"


def test_the_converter_is_for_one_interpreter():
    """Its file carries this interpreter's tag, so another Python version does not load it and goes through ctypes."""
    name = os.path.basename(_build.PYCALL)
    suffixes = importlib.machinery.EXTENSION_SUFFIXES
    assert name == "_pycall" + suffixes[0]
    assert suffixes[0] not in (".so", ".abi3.so")
