"""Compile the HIP sources under csrc/ for gfx950 into libmxfp4_hip.so, and the native host path of the Python front
ends (csrc/mx_torch.cpp, against the installed torch) into _mx_torch.so, both in-tree."""
import os
import subprocess
import sys

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libmxfp4_hip.so")
SOURCES = ["mx_api.hip", "mx_quant.hip", "mx_gemm.hip", "mx_optim.hip"]
HEADERS = ["mx_device.hpp", "mx_launch.hpp", os.path.join("..", "..", "include", "mxfp4.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]

HOST_SOURCE, HOST_LIB = "mx_torch.cpp", os.path.join(_HERE, "_mx_torch.so")


def host_command():
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-DTORCH_EXTENSION_NAME=_mx_torch", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
            os.path.join(CSRC, HOST_SOURCE), "-o", HOST_LIB, "-L" + _HERE, "-l:libmxfp4_hip.so", "-Wl,-rpath,$ORIGIN",
            "-L" + os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python", "-lc10_hip"]


def is_stale():
    if not os.path.exists(LIB) or not os.path.exists(HOST_LIB):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(HOST_LIB))
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS + [HOST_SOURCE]]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force=True, verbose=False, extra_flags=()):
    """Build the two shared libraries; returns the HIP library's path."""
    if not force and not is_stale():
        return LIB
    cmd = [HIPCC] + FLAGS + list(extra_flags) + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    cmd = host_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build(force=True, verbose=True, extra_flags=sys.argv[1:])
    print(LIB)
