"""Build libcacnn.so (host planner + gfx950 kernels) with hipcc and _cacnn_torch.so (the binding's calls on torch tensors) with the host
compiler, in-tree.  Usage: python paper_1802_06905_amd/build.py"""
import os
import shutil
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcacnn.so")
SOURCES = ["cacnn_host.cpp", "cacnn_kernels.hip", "cacnn_flat.hip", "cacnn_window.hip", "cacnn_pool.hip", "cacnn_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

TORCH_LIB = os.path.join(HERE, "_cacnn_torch.so")


def torch_command() -> list:
    """How _cacnn_torch.so is compiled: torch's own headers and libraries, which are in the process before it is imported."""
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(shutil.which(HIPCC) or HIPCC))        # (HIPCC may be a name that PATH finds)
    return [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", os.path.join(root, "include"),
            "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"), "-o", TORCH_LIB,
            os.path.join(CSRC, "cacnn_torch.cpp"), "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link the shared library, and the module beside it.  Always recompiles.  Without the module (its
    compiler or torch's headers fail: a warning) the binding's calls take a longer way; an old one, made for another library, is removed."""
    cmd = [HIPCC] + FLAGS + ["-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    if os.path.exists(TORCH_LIB):
        os.remove(TORCH_LIB)
    beside, torch_out = None, ""
    try:
        torch_cmd = torch_command()
        if verbose:
            print(" ".join(torch_cmd))
        beside = subprocess.Popen(torch_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except (ImportError, OSError) as error:
        torch_out = str(error)
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if beside is not None:
        torch_out = beside.communicate()[0]
    # the host pass does not know the packed-fp32 feature and says so once per file: not an error
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    if beside is None or beside.returncode != 0:
        warnings.warn(f"{os.path.basename(TORCH_LIB)} was not built, calls of the binding take a longer way:\n{torch_out}", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
