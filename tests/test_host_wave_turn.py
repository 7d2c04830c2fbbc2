"""The M <= 64 kernel's lane exchange through LDS (csrc/fq_turn.h) must not rest on the order in which a compiler happens to leave
a lane's own reads and writes: run on the host with the lanes as far apart as the source lets them be."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_20839_amd", "csrc")
CLANG = shutil.which("clang++", path=os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin"))


@pytest.mark.skipif(CLANG is None, reason="needs the ROCm clang (vector types)")
def test_lanes_read_what_the_others_wrote(tmp_path):
    exe = str(tmp_path / "wave_turn_check")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "host", "wave_turn_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "wrong bytes 0" in out.stdout, out.stdout
