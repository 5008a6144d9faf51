"""Builds libosc.so (the product) and libosc_probe.so (the benchmark's matrix-core yardstick) in-tree
with hipcc, for gfx950 only, and _native.so, the host code of the Python binding's per-step calls."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libosc.so")
PROBE_LIB = os.path.join(HERE, "libosc_probe.so")
SOURCES = ["api.hip", "tuning.hip", "quant.hip", "gemm.hip", "gemm_flow.hip", "profile.hip", "fused.hip", "g16.hip"]
PROBE_SOURCES = ["probe.hip"]
NATIVE = os.path.join(HERE, "_native.so")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _native_command():
    import torch
    from torch.utils.cpp_extension import include_paths
    root = os.path.dirname(torch.__file__)
    inc = [f"-isystem{p}" for p in include_paths()] + [f"-I{sysconfig.get_paths()['include']}", "-isystem/opt/rocm/include"]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc, os.path.join(CSRC, "native.cpp"), "-o", NATIVE,
            f"-L{os.path.join(root, 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", f"-L{HERE}", "-l:libosc.so",
            "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{os.path.join(root, 'lib')}"]


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for s in SOURCES + PROBE_SOURCES:
        o = os.path.join(CSRC, s.replace(".hip", ".o"))
        objs.append(o)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    for s, p in procs:
        out = p.communicate()[0].decode()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {s}:\n{out}")
        if verbose and out.strip():
            print(out)
    n = len(SOURCES)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs[:n], "-o", LIB])
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs[n:], "-o", PROBE_LIB])
    cmd = _native_command()  # links libosc.so, so it comes last
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
