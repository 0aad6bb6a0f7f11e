"""Builds the HIP library in-tree, paper_2505_24034_amd/libllamarl.so (gfx950 only), and the binding's argument
marshalling, _native.so (host code against torch's headers)."""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libllamarl.so")
SOURCES = ["llamarl.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
    # keep hipcc from forming packed-fp32 VALU ops out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]
NATIVE_PATH = os.path.join(HERE, "_native.so")
CXX = os.environ.get("CXX", "g++")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "is not a recognized feature for this target" not in l)
    if verbose and out.strip():
        print(out, flush=True)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), out))


def build_library(verbose=True, extra_flags=()):
    _run([HIPCC] + FLAGS + list(extra_flags) + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB_PATH], verbose)
    build_native(verbose)
    return LIB_PATH


def rocm_root():
    """the ROCm installation of the compiler in use, which may be given by name alone"""
    return os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC) or HIPCC)))


def build_native(verbose=True):
    """csrc/native.cpp; needs libllamarl.so"""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               os.path.join(rocm_root(), "include"), sysconfig.get_paths()["include"]]
    cmd = [CXX, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    for d in include:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "native.cpp"), "-o", NATIVE_PATH, "-L" + os.path.join(root, "lib"), "-ltorch", "-ltorch_cpu",
            "-ltorch_python", "-lc10", "-lc10_hip", "-ltorch_hip", "-L" + HERE, "-l:libllamarl.so", "-Wl,-rpath,$ORIGIN"]
    _run(cmd, verbose)
    return NATIVE_PATH


if __name__ == "__main__":
    build_library(extra_flags=sys.argv[1:])
