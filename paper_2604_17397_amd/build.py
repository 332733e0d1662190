"""Compile the HIP sources under csrc/ into libsdvg.so (gfx950) next to this file, and the argument
marshalling under csrc/host/ into the extension module _native.so."""
import glob
import os
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsdvg.so")
NATIVE = os.path.join(HERE, "_native.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed fp32 instructions (v_pk_*_f32)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]
# Sources compiled with a kernel's first dwords of arguments (14 at most) preloaded into scalar registers: worth 0.3 us
# of a launch where the arguments are what a short kernel waits for. The routers lose 0.2 us by it.
PRELOADED = {"block_attn_rows32.hip", "rope.hip"}
PRELOAD_FLAGS = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False, extra_flags=(), out: str = LIB) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [*HIPCC_FLAGS, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def run(args):
        cmd = [hipcc, *flags, *args]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        noise = "is not a recognized feature for this target"
        log = "\n".join(ln for ln in res.stdout.splitlines() if noise not in ln)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + log)
        if verbose and log.strip():
            print(log)
        return log

    def compile_one(src, obj):
        return run([*(PRELOAD_FLAGS if os.path.basename(src) in PRELOADED else []), "-c", src, "-o", obj])

    with tempfile.TemporaryDirectory(prefix="sdvg_build_") as tmp, ThreadPoolExecutor(4) as pool:
        objects = [os.path.join(tmp, os.path.basename(src) + ".o") for src in sources()]
        logs = list(pool.map(compile_one, sources(), objects))
        logs.append(run([*objects, "-o", out]))
    return "\n".join(log for log in logs if log)


def build_native(verbose: bool = False, out: str = NATIVE) -> str:
    import torch
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"]]
    for path in cpp_extension.include_paths():
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "host", "native.cpp"), "-o", out]
    for path in cpp_extension.library_paths():
        cmd += ["-L", path]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("native module failed to build:\n" + res.stdout)
    if verbose and res.stdout.strip():
        print(res.stdout)
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra_flags=sys.argv[1:]))
    print(build_native(verbose=True))
