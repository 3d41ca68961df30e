"""Build the native libraries in-tree: the HIP attention library (hipcc for gfx950) into
paper_2608_26523_amd/libvpp_chunk_attn.so, the host-only schedule model (g++) into
paper_2608_26523_amd/libvpp_sched.so, and the extension that calls the attention library on
torch tensors (g++) into paper_2608_26523_amd/vpp_torch.so."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "vpp_chunk_attn.hip")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libvpp_chunk_attn.so")
SCHED_SRC = os.path.join(PKG, "csrc", "vpp_sched.cpp")
SCHED_LIB = os.path.join(PKG, "libvpp_sched.so")
TORCH_SRC = os.path.join(PKG, "csrc", "vpp_torch.cpp")
TORCH_LIB = os.path.join(PKG, "vpp_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-shared",
    # no packed fp32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


PARTS = (0, 1, 2)  # VPP_PART values: host code + contiguous-cache kernels, paged, split-key


def build(extra_flags=(), out: str = LIB, quiet: bool = True, src: str = None) -> str:
    """Compile the parts of the HIP source in parallel (one hipcc each), then link."""
    src = src or SRC
    base = [hipcc()] + HIPCC_FLAGS + list(extra_flags) + ["-I", INCLUDE]
    objs = [out + ".part%d.o" % part for part in PARTS]
    procs = []
    for part, obj in zip(PARTS, objs):
        cmd = [c for c in base if c != "-shared"] + ["-c", "-DVPP_PART=%d" % part, "-o", obj, src]
        procs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    outs = [pr.communicate()[0] for pr in procs]
    msgs = [ln for o in outs for ln in o.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if any(pr.returncode != 0 for pr in procs):
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    tmp = out + ".tmp"
    res = subprocess.run(base + ["-o", tmp] + objs, capture_output=True, text=True)
    msgs += [ln for ln in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    for obj in objs:
        if os.path.exists(obj):
            os.remove(obj)
    if res.returncode != 0:
        raise RuntimeError("hipcc link failed:\n" + "\n".join(msgs))
    if msgs and not quiet:
        print("\n".join(msgs), file=sys.stderr)
    os.replace(tmp, out)
    return out


def build_sched(out: str = SCHED_LIB) -> str:
    """The schedule model is plain host C++: no HIP, so it loads on any machine."""
    tmp = out + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-I", INCLUDE, "-o", tmp, SCHED_SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, out)
    return out


def build_torch(out: str = TORCH_LIB) -> str:
    """The extension module is host C++ against torch's headers; it runs no kernel of its own."""
    import sysconfig

    import torch
    troot = os.path.dirname(torch.__file__)
    tlib = os.path.join(troot, "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = out + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I", INCLUDE, "-isystem", os.path.join(troot, "include"),
           "-isystem", os.path.join(troot, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"),
           "-o", tmp, TORCH_SRC, "-L", tlib, "-Wl,-rpath," + tlib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch",
           "-ltorch_python"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(quiet=False))
    print(build_sched())
    print(build_torch())
