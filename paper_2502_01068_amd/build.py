"""Build libfastkv_select.so for gfx950 with hipcc (cross-compiles without a GPU) and the binding's native
call path (_native.so) with the host compiler."""
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libfastkv_select.so")
NATIVE = os.path.join(PKG, "_native.so")
SOURCES = ["fkv_api.hip", "fkv_score.hip", "fkv_score_fused.hip", "fkv_score_keep.hip", "fkv_select.hip", "fkv_select_gather.hip", "fkv_select_long.hip", "fkv_select_coop.hip", "fkv_gather.hip", "fkv_decode.hip", "fkv_diag.hip", "fkv_probe.hip", "fkv_wout.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build(verbose: bool = False, extra=()) -> str:
    cmd = [HIPCC, *FLAGS, *extra, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB + ".tmp"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(LIB + ".tmp", LIB)
    return LIB


def build_native() -> str:
    """The CPython extension between torch tensors and the C ABI; no GPU code, no link to the library."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-I" + os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"]]
    for path in cpp_extension.include_paths("cuda"):
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "fkv_torch.cpp"), "-o", NATIVE + ".tmp", "-L" + lib_dir,
            "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("host compiler failed:\n" + res.stdout)
    os.replace(NATIVE + ".tmp", NATIVE)
    return NATIVE


if __name__ == "__main__":
    import sys
    print(build(verbose=True, extra=sys.argv[1:]))
    print(build_native())
