"""Build the HIP library (gfx950) into paper_2605_12245_amd/libsoar_hip.so, and the marshalling module soar_host.so beside it."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "soar_hip.hip")
OUT = os.path.join(HERE, "libsoar_hip.so")
HOST_SRC = os.path.join(HERE, "csrc", "soar_host.cpp")
HOST_OUT = os.path.join(HERE, "soar_host.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: the kernels state every fused multiply-add explicitly; the
# compiler must not form others.  No fast-math: IEEE division, subnormals kept.
# Packed-FP32 instructions are disabled for device code.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"),
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = [l for l in r.stdout.splitlines()
             if l.strip() and "is not a recognized feature for this target" not in l]
    if r.returncode != 0 or verbose:
        print("\n".join(lines))
    if r.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed")


def build_host(verbose: bool = False) -> str:
    import torch
    at = os.path.dirname(torch.__file__)
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
          "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(at, "include"), "-isystem", sysconfig.get_paths()["include"],
          HOST_SRC, "-o", HOST_OUT, "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"], verbose)
    return HOST_OUT


def build(verbose: bool = False, extra=()) -> str:
    _run([HIPCC, *FLAGS, *extra, SRC, "-o", OUT], verbose)
    build_host(verbose)
    return OUT


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
