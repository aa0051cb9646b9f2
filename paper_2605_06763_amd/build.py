"""Compile the HIP sources under csrc/ into one in-tree shared library for gfx950, and the Python module that calls it."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB_PATH = os.path.join(_HERE, "liblouver.so")
# the Python module of the decode loop's calls (csrc/pycall.cpp, host code only); another Python does not find it by this name
CALL_PATH = os.path.join(_HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJ_DIR = os.path.join(_HERE, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the leading scalar arguments of a kernel arrive in registers with the dispatch (kernels order theirs accordingly)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd: list[str]) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compiler failed: " + " ".join(cmd) + "\n" + res.stdout + res.stderr)
    return res.stderr


def _call_command(out: str) -> list[str]:
    """The host compiler's line for the Python module: torch's headers, nothing of the GPU."""
    import torch
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-isystem" + p for p in cpp_extension.include_paths()]
    cmd += [os.path.join(CSRC, "pycall.cpp"), "-o", out]
    return cmd + ["-L" + p for p in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"]


def build_call_module(path: str = CALL_PATH) -> str:
    """The Python module, put in place whole.  Without a host compiler or torch's headers there is none: every call goes
    through ctypes then, some 3 to 5 us slower on the host."""
    part = path + ".part"
    try:
        log = _run(_call_command(part))
        os.replace(part, path)
        return log
    except (OSError, RuntimeError, ImportError) as e:
        for p in (part, path):   # nor one that was built for other sources
            if os.path.exists(p):
                os.remove(p)
        warnings.warn(f"{os.path.basename(path)} was not built, calls go through ctypes: {e}")
        return ""


def build_library(verbose: bool = False, jobs: int | None = None) -> str:
    """One object per source (compiled side by side), then one link."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(OBJ_DIR, os.path.basename(s)[:-4] + ".o") for s in srcs]
    jobs = jobs or min(len(srcs), os.cpu_count() or 1, 16)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        call = pool.submit(build_call_module)
        logs = list(pool.map(lambda so: _run([hipcc, *HIPCC_FLAGS, "-c", so[0], "-o", so[1]]), zip(srcs, objs)))
        logs.append(call.result())
    logs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]))
    if verbose:
        # the host pass does not know the packed-fp32 feature name and says so; that is expected
        print("\n".join(l for log in logs for l in log.splitlines() if "packed-fp32-ops" not in l))
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
