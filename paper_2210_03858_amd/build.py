"""Builds libbcq_hip.so (HIP kernels + C ABI) for gfx950 with hipcc and _bcq_torch.so (host path of the hot entry
points and the autograd node, linked against it), in-tree.

Usage: python -m paper_2210_03858_amd.build        (always recompiles)
"""
import concurrent.futures
import glob
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbcq_hip.so")
TORCH_LIB = os.path.join(HERE, "_bcq_torch.so")
BUILD_DIR = os.path.join(HERE, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-ffp-contract=off",
    # packed-fp32 instructions stay off for all device code of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc():
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _torch_commands():
    """(compile, link) command of the torch extension; its object file lies beside the kernels'."""
    from torch.utils import cpp_extension
    import torch
    obj = os.path.join(BUILD_DIR, "bcq_torch.o")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(_hipcc())))
    include = [os.path.join(os.path.dirname(torch.__file__), "include")]
    include += [os.path.join(include[0], "torch", "csrc", "api", "include"), os.path.join(rocm, "include"),
                sysconfig.get_paths()["include"]]
    libs = ["-L" + d for d in cpp_extension.library_paths()]
    libs += ["-ltorch", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    compile_cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                   "-DTORCH_EXTENSION_NAME=_bcq_torch", "-DTORCH_API_INCLUDE_EXTENSION_H",
                   "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    compile_cmd += [a for d in include for a in ("-isystem", d)]
    compile_cmd += ["-c", os.path.join(CSRC, "bcq_torch.cpp"), "-o", obj]
    link_cmd = ["g++", "-shared", "-fPIC", obj, "-L" + HERE, "-lbcq_hip", "-Wl,-rpath,$ORIGIN"] + libs
    return compile_cmd, link_cmd


def build_library(verbose=False):
    os.makedirs(BUILD_DIR, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    torch_compile, torch_link = _torch_commands()
    objs = [os.path.join(BUILD_DIR, os.path.basename(s)[:-4] + ".o") for s in sources]

    def compile_one(cmd):
        return subprocess.run(cmd, capture_output=True, text=True)

    commands = [[_hipcc()] + HIPCC_FLAGS + ["-c", src, "-o", obj] for src, obj in zip(sources, objs)] + [torch_compile]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(commands))) as ex:
        for cmd, r in zip(commands, ex.map(compile_one, commands)):
            if verbose and r.stderr.strip():
                print(r.stderr)
            if r.returncode != 0:
                raise RuntimeError("failed: %s\n%s" % (" ".join(cmd), r.stderr))
    tmp = LIB + ".%d.tmp" % os.getpid()
    r = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stderr)
    os.replace(tmp, LIB)
    tmp = TORCH_LIB + ".%d.tmp" % os.getpid()
    r = subprocess.run(torch_link + ["-o", tmp], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stderr)
    os.replace(tmp, TORCH_LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
