"""Builds the HIP library in-tree: ``csrc/*.hip`` -> ``paper_2505_20839_amd/libfireq.so`` (gfx950), and the binding's
argument marshalling: ``csrc/fq_marshal.cpp`` -> ``paper_2505_20839_amd/_fq_marshal-*.so`` (host code, a Python extension)."""
from __future__ import annotations

import glob
import hashlib
import os
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libfireq.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-result",
    # packed FP32 VALU forms are kept off for this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_library(verbose: bool = False) -> str:
    """Compile every kernel for gfx950 and link the shared library.  Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB_PATH + ".tmp%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + sources() + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


def marshal_path() -> str:
    """Where the argument marshalling is, or will be, built.  It calls the library through bare addresses, so the name carries a
    digest of what decides the arguments of those calls and the binary interface it was compiled against: its source, the C
    declarations, torch and Python."""
    import sysconfig

    import torch
    include = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")
    digest = hashlib.sha256()
    for path in (os.path.join(CSRC, "fq_marshal.cpp"), os.path.join(include, "fireq.h"), os.path.join(include, "fireq_kv4_ws.h"),
                 os.path.join(include, "fireq_wquant_ws.h")):
        with open(path, "rb") as f:
            digest.update(f.read())
    digest.update(repr((torch.__version__, sysconfig.get_config_var("EXT_SUFFIX"))).encode())
    return os.path.join(PKG_DIR, "_fq_marshal-%s.so" % digest.hexdigest()[:16])


def build_marshal() -> str:
    """Compile the argument marshalling against the installed torch and Python.  Always recompiles."""
    import sysconfig

    import torch
    path = marshal_path()
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = path + ".tmp%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", inc, "-isystem",
           os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
           "-isystem", os.path.join(rocm, "include"), os.path.join(CSRC, "fq_marshal.cpp"), "-o", tmp,
           "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("g++ failed:\n" + res.stdout)
    os.replace(tmp, path)
    for old in glob.glob(os.path.join(PKG_DIR, "_fq_marshal*.so")):
        if old != path:
            os.remove(old)
    return path


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
    print(build_marshal())
