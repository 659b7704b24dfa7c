"""Build libadahop.so (HIP, gfx950 only) in-tree with hipcc, and the binding's native half with g++.  No GPU is needed to compile."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libadahop.so")
CALL = os.path.join(HERE, "_call.so")
SOURCES = ["api.hip", "quantize.hip", "foid.hip", "gemm_mx.hip", "gemm_mx_dual.hip", "gemm_mx_small.hip", "oe_bf16.hip", "pattern.hip", "oht.hip", "probe.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-ffp-contract=off", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument"]


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def call_command():
    """The command that builds csrc/call.cpp, a Python module against torch's own headers and libraries."""
    import torch
    from torch.utils import cpp_extension
    root = os.path.dirname(torch.__file__)
    include = [f"-I{p}" for p in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]]
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
            + include + [os.path.join(CSRC, "call.cpp"), "-o", CALL, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"])


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared libraries; always recompiles."""
    objs = []
    procs = [("call.cpp", subprocess.Popen(call_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))]
    for s in SOURCES:
        obj = os.path.join(CSRC, s.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc()] + FLAGS + ["-c", os.path.join(CSRC, s), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if out.strip() and (verbose or p.returncode != 0):
            print(out, file=sys.stderr, flush=True)
        failed |= p.returncode != 0
    if failed:
        raise RuntimeError("a source does not compile")
    subprocess.run([hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
