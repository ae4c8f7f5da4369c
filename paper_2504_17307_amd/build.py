"""Compile the HIP library for gfx950 with hipcc (cross-compiles without a GPU)."""
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
SRC = os.path.join(CSRC, "uccl_chunk.hip")  # the one translation unit; it includes the .hpp files beside it
INC = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libuccl_chunk.so")
# aids of bench.py (dense streaming kernels) and of the tests (the report's recount, late decisions), a library of their own
PROBE_SRC = [os.path.join(PKG, "probe", f) for f in ("stream_probe.hip", "report_probe.hip", "group_probe.hip", "late_probe.hip")]
PROBE_LIB = os.path.join(PKG, "probe", "libuccl_probe.so")

# prepared calls of the Python binding: a CPython extension, host code only, for the interpreter that builds it
PREPARED_SRC = os.path.join(CSRC, "prepared_call.c")
PREPARED_LIB = os.path.join(PKG, "_prepared" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fno-fast-math", "-ffp-contract=off", "-fno-gpu-flush-denormals-to-zero",
    # keep packed fp32 VALU forms out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
]


def sources():
    """Every file the library is built from (kernel sources and the public header)."""
    files = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".hpp")))
    return files + [os.path.join(INC, "uccl_chunk.h")]


def build(extra_flags=(), out=LIB, verbose=False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = out + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, f"-I{INC}", f"-I{CSRC}", SRC, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


def build_probe(verbose=False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = PROBE_LIB + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIPCC_FLAGS, f"-I{INC}", f"-I{CSRC}", *PROBE_SRC, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, PROBE_LIB)
    return PROBE_LIB


def build_prepared(verbose=False) -> str:
    tmp = PREPARED_LIB + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-shared", "-fPIC", "-Wall", "-Wextra", "-Wno-missing-field-initializers", "-Wno-cast-function-type",
           "-I" + sysconfig.get_paths()["include"], PREPARED_SRC, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, PREPARED_LIB)
    return PREPARED_LIB


if __name__ == "__main__":
    print(build(sys.argv[1:], verbose=True))
    print(build_probe(verbose=True))
    print(build_prepared(verbose=True))
