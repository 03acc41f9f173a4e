"""The native part of the binding is an addition: without it, or with one for another torch, calls go through ctypes."""
import os
import subprocess
import sys

import pytest

import paper_2502_00527_amd as pq
from paper_2502_00527_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

needs_library = pytest.mark.skipif(not os.path.exists(pq.lib_path()), reason="libpolarquant.so is not built")


@needs_library
def test_calls_are_made_without_the_native_part(monkeypatch):
    def missing(*args):
        raise ImportError("No module named _native")

    monkeypatch.setattr(pq, "_calls", None)
    monkeypatch.setattr(pq.importlib, "import_module", missing)
    torch = pytest.importorskip("torch")
    layout = pq.Layout(128, 4, 4, 128, 2, 0)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        with pytest.raises(pq.PolarQuantError, match="device tensor"):      # the ctypes way's own check
            pq.pq_encode_keys(layout, torch.zeros(128, 2, 128), None, None, None)
    for name in ("decode_attention", "score_keys", "encode_keys", "encode_values", "append_keys"):
        assert getattr(pq._calls, name)(1, 2, 3) is None


@needs_library
@pytest.mark.skipif(not os.path.exists(build.BINDING_PATH), reason="the native part is not built")
@pytest.mark.parametrize("version", [None, "0.0.1"])
def test_the_native_part_is_for_one_torch(version):
    code = "import torch, warnings\n" + (f"torch.__version__ = {version!r}\n" if version else "") + \
        "warnings.simplefilter('error')\nimport paper_2502_00527_amd as pq\nprint(type(pq._marshaller()).__name__)"
    run = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    if version is None:
        assert run.returncode == 0 and run.stdout.strip() == "module", run.stderr
    else:
        assert run.returncode != 0 and "built for torch" in run.stderr, run.stderr


def test_the_library_builds_without_what_the_native_part_needs(monkeypatch):
    assert build.binding_lacks() is None
    assert os.path.basename(build.BINDING_PATH).startswith("_native.") and "cpython" in build.BINDING_PATH
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.binding_lacks() == "g++"
    monkeypatch.undo()
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": "/nowhere"})
    assert "Python.h" in build.binding_lacks()
