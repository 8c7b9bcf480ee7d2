"""Builds libpk.so (the C-ABI library with the gfx950 kernels) and the CPython binding of its op calls in-tree with hipcc."""
import hashlib
import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libpk.so")
CALL_PATH = os.path.join(HERE, "_pk_call.so")
CSRC = os.path.join(HERE, "csrc")
SOURCES = [os.path.join(CSRC, n) for n in ("pk_kernels.hip", "gemm_rs.hip", "gemm_rs16.hip", "gemm_ag.hip", "gemm_agk.hip")]
HEADERS = [os.path.join(CSRC, n) for n in ("pk_device.h", "pk_gemm.h", "pk_tiles.h")] + [
    os.path.join(os.path.dirname(HERE), "include", "pk.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Werror=division-by-zero",
    # packed-fp32 VALU forms are kept off for every HIP source of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def header_digest():
    """What tells the interface that a library and an extension module were compiled with from another one."""
    with open(HEADERS[-1], "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def build_library(verbose=False):
    """Compile libpk.so; always recompiles (the sources side by side).  Returns the path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        digest = '-DPK_HEADER_DIGEST="%s"' % header_digest()
        cmds = [[hipcc] + HIPCC_FLAGS + [digest, "-c", s, "-o", o] for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(max_workers=min(8, len(cmds))) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        _run([hipcc] + HIPCC_FLAGS + ["-shared"] + objs + ["-o", LIB_PATH], verbose)
    return LIB_PATH


def _run(cmd, verbose):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed building libpk.so")


def build_binding(verbose=False):
    """Compile csrc/pk_call.cpp (host code only) against torch."""
    import torch
    from torch.utils import cpp_extension
    from . import pk
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    include = [sysconfig.get_path("include")] + cpp_extension.include_paths("cuda")
    _run([hipcc, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DPK_BUILT_FOR="%s"' % pk.built_for(header_digest())] +
         ["-isystem" + i for i in include] +
         [os.path.join(CSRC, "pk_call.cpp"), "-L", os.path.join(os.path.dirname(torch.__file__), "lib"),
          "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-o", CALL_PATH], verbose)
    return CALL_PATH


C_LAUNCH_SRC = os.path.join(os.path.dirname(HERE), "tests", "c_abi_launch.c")
C_LAUNCH_LIB = os.path.join(os.path.dirname(HERE), "tests", "libc_abi_launch.so")


def build_c_launch_check():
    """Compile the plain-C caller of the library (tests/c_abi_launch.c) with gcc as a shared object that the GPU tests
    load: it sees include/pk.h and the HIP runtime's C interface only."""
    gcc = os.environ.get("CC", "gcc")
    cmd = [gcc, "-std=c99", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(os.path.dirname(HERE), "include"),
           "-I", "/opt/rocm/include", C_LAUNCH_SRC, "-L", HERE, "-l:libpk.so", "-L/opt/rocm/lib", "-lamdhip64",
           "-Wl,-rpath,$ORIGIN/../paper_2511_13940_amd", "-Wl,-rpath,/opt/rocm/lib", "-o", C_LAUNCH_LIB]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        raise RuntimeError("gcc failed building tests/libc_abi_launch.so")
    return C_LAUNCH_LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_binding(verbose=True))
    print(build_c_launch_check())
