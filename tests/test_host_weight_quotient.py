"""The weight quantiser's short quotient (one multiply and two FMAs with the group scale's reciprocal) must round to the
same integer as an IEEE division, for every weight and every E4M3 scale.  The model runs the same FP32 operations on the
host (C, hardware FMA)."""
import os
import shutil
import subprocess

import pytest

from test_host_fast_quotient import _cpu_has_fma

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "weight_quotient_check.c")


@pytest.mark.skipif(shutil.which("gcc") is None or not _cpu_has_fma(), reason="needs gcc and a CPU with FMA")
def test_short_quotient_rounds_to_the_ieee_code(tmp_path):
    exe = str(tmp_path / "weight_quotient_check")
    subprocess.run(["gcc", "-O2", "-mfma", "-fopenmp", "-ffp-contract=off", SRC, "-o", exe, "-lm"], check=True)
    # every 3rd x (2.9e8 quotients); FQ_EXHAUSTIVE=1 runs all of them
    out = subprocess.run([exe, "1" if os.environ.get("FQ_EXHAUSTIVE") else "3"], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert "code differences 0" in out.stdout


@pytest.mark.skipif(shutil.which("gcc") is None or not _cpu_has_fma(), reason="needs gcc and a CPU with FMA")
def test_short_divisions_of_the_group_scale_are_the_ieee_quotients(tmp_path):
    """max / 7 for every significand, 1 / sigma8 for every E4M3 significand from any estimate within one unit."""
    exe = str(tmp_path / "weight_scale_check")
    src = os.path.join(os.path.dirname(SRC), "weight_scale_check.c")
    subprocess.run(["gcc", "-O2", "-mfma", "-ffp-contract=off", src, "-o", exe, "-lm"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and "differences 0" in out.stdout, out.stdout
