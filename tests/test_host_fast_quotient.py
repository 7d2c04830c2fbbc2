"""The activation quantiser's short quotient (one multiply and two FMAs with the row's reciprocal)
must store the same E4M3 code as an IEEE division, for every input the kernel can see.  The model
below runs the same FP32 operations on the host (C, hardware FMA) over the whole input domain."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host", "activation_quotient_check.c")


def _cpu_has_fma():
    try:
        return " fma " in open("/proc/cpuinfo").read().replace("\n", " ")
    except OSError:
        return False


@pytest.mark.skipif(shutil.which("gcc") is None or not _cpu_has_fma(), reason="needs gcc and a CPU with FMA")
def test_scale_reciprocal_and_signed_quotient_are_the_ieee_ones(tmp_path):
    """Scale and reciprocal without a division, and the codes with the sign of zero."""
    exe = str(tmp_path / "activation_quotient_check")
    subprocess.run(["gcc", "-O2", "-mfma", "-fopenmp", "-ffp-contract=off", SRC, "-o", exe, "-lm"], check=True)
    # every 3rd absmax (1.8e8 pairs, a few seconds); FQ_EXHAUSTIVE=1 runs all 5.3e8
    out = subprocess.run([exe, "1" if os.environ.get("FQ_EXHAUSTIVE") else "3"], capture_output=True, text=True)
    assert out.returncode == 0 and "differences 0" in out.stdout, out.stdout
