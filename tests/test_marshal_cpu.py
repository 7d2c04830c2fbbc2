"""The binding without its native argument marshalling, and which built extension it takes (no kernel is launched here)."""
import types

import pytest

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
    unbound.setattr(build, "MARSHAL_PATH", str(tmp_path / "absent.so"))
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
    unbound.setattr(build, "MARSHAL_PATH", str(broken))
    with pytest.warns(RuntimeWarning, match="broken.so"):
        assert binding.fq_w4a8_gemm_workspace_bytes(513, 256, 4096) == 2 * 4 * 513 * 16


def test_the_built_extension_is_taken(unbound):
    assert isinstance(binding.marshal(), types.ModuleType)
    assert binding.marshal().gemm_workspace_bytes(513, 256, 4096) == 2 * 4 * 513 * 16
