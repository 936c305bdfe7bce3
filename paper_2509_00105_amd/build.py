"""Build the HIP library (libkvh.so) in-tree for gfx950 with hipcc, and the binding's call module (_fastcall) with the C++ compiler."""
from __future__ import annotations

import os
import shlex
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libkvh.so")
CALLS = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))  # for the interpreter that builds it alone
SOURCES = ["kvh_api.hip", "kvh_decode.hip", "kvh_encode.hip", "kvh_transcode.hip", "kvh_loader.hip", "kvh_policy.cpp"]

# -ffp-contract=off: the codec's arithmetic fuses only where the source says fma.
# -fno-honor-nans: inputs are finite by contract; without it every min/max of a value unpacked with
# integer ops is preceded by a canonicalising v_max (sNaN quieting).
# packed-fp32-ops off: hipcc must not form v_pk_*_f32 from the scalar float code.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-honor-nans",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _compile(target: str, cmd: list, verbose: bool) -> None:
    """Run cmd with the output file appended and put the result in place of target."""
    tmp = target + ".tmp.%d" % os.getpid()
    res = subprocess.run([*cmd, "-o", tmp], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = "is not a recognized feature for this target"
    out = "\n".join(ln for ln in res.stdout.splitlines() if noise not in ln)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))
    if verbose and out.strip():
        print(out)
    os.replace(tmp, target)


def _build_calls(verbose: bool) -> None:
    """The call module makes calls cheaper and is no part of what they need: without Python's headers or a C++ compiler it is
    left out, and the binding goes through ctypes."""
    for old in (CALLS, os.path.join(HERE, "_fastcall.so")):  # none is left that does not belong to this library
        if os.path.exists(old):
            os.remove(old)
    include, cxx = sysconfig.get_paths()["include"], shlex.split(os.environ.get("CXX", "g++"))
    if not os.path.exists(os.path.join(include, "Python.h")) or not cxx or shutil.which(cxx[0]) is None:
        print("no Python.h or no C++ compiler: calls go through ctypes")
        return
    _compile(CALLS, [*cxx, "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", include, os.path.join(CSRC, "kvh_fastcall.cpp")], verbose)


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _compile(LIB, [hipcc, *HIPCC_FLAGS, *[os.path.join(CSRC, s) for s in SOURCES]], verbose)
    _build_calls(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
