"""The binding without its native argument marshalling, and which built extension it takes (no kernel is launched here)."""
import os
import shutil
import types

import pytest
import torch

from paper_2505_20839_amd import binding, build


@pytest.fixture
def unbound(monkeypatch):
    """The binding as a fresh process has it: no marshalling looked for yet."""
    monkeypatch.setattr(binding, "_marshal", None)
    return monkeypatch


def _fails():
    raise RuntimeError("no compiler here")


def test_calls_work_without_the_extension(unbound, tmp_path):
    """No extension and none to be had (no compiler, no headers): one warning, then every call takes its Python form."""
    unbound.setattr(build, "marshal_path", lambda: str(tmp_path / "absent.so"))
    unbound.setattr(build, "build_marshal", _fails)
    with pytest.warns(RuntimeWarning, match="no compiler here") as seen:
        assert binding.fq_w4a8_gemm_workspace_bytes(2048, 4096, 11008) == 2 * 12 * 2048 * 16
        assert binding.fq_w4a8_gemm_workspace_bytes(64, 256, 4096) == 0
        with pytest.raises(TypeError, match="X must be a GPU tensor"):
            binding.fq_quantize_act(None)
        with pytest.raises(TypeError, match="P must be a GPU tensor"):
            binding.fq_kv4_output(None, None, None, None)
    assert len(seen) == 1


def test_calls_work_with_an_extension_that_does_not_load(unbound, tmp_path):
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"not a library")
    unbound.setattr(build, "marshal_path", lambda: str(broken))
    with pytest.warns(RuntimeWarning, match="broken.so"):
        assert binding.fq_w4a8_gemm_workspace_bytes(513, 256, 4096) == 2 * 4 * 513 * 16


def test_the_built_extension_is_taken(unbound):
    assert isinstance(binding.marshal(), types.ModuleType)
    assert binding.marshal().gemm_workspace_bytes(513, 256, 4096) == 2 * 4 * 513 * 16


@pytest.mark.parametrize("change", ["source", "header", "torch"])
def test_an_extension_of_other_sources_is_not_bound(unbound, tmp_path, change):
    """An extension built from another state of its source, of the C declarations, or against another torch takes other
    arguments than the library's functions: it is built anew, never bound (here, where that fails, the Python forms run)."""
    for sub in ("paper_2505_20839_amd/csrc", "include"):
        shutil.copytree(os.path.join(os.path.dirname(build.PKG_DIR), sub), tmp_path / sub)
    unbound.setattr(build, "CSRC", str(tmp_path / "paper_2505_20839_amd" / "csrc"))
    if change == "torch":
        unbound.setattr(torch, "__version__", "0.0")
    else:
        name = "paper_2505_20839_amd/csrc/fq_marshal.cpp" if change == "source" else "include/fireq_kv4_ws.h"
        (tmp_path / name).write_text((tmp_path / name).read_text() + "\n")
    unbound.setattr(build, "build_marshal", _fails)
    with pytest.warns(RuntimeWarning, match="no compiler here"):
        binding.marshal()
