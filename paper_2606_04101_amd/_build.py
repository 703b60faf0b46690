"""Build libultraep.so (hipcc, gfx950) and the native half of the Python binding
(_native.so, the host compiler) in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libultraep.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["abi.hip", "count.hip", "plan.hip", "dispatch.hip", "pack.hip",
           "relay.hip", "combine.hip", "reduce.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         # packed fp32 instructions are disabled for all device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# the fp32 steps round every product and sum on its own: no contraction into
# fused multiply-adds (the other sources have no fp32 arithmetic to fuse)
EXTRA = {"combine.hip": ["-ffp-contract=off"], "reduce.hip": ["-ffp-contract=off"]}


def build_native() -> str:
    """csrc/binding.cpp against torch's headers and libraries."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f'-DTORCH_BUILD="{torch.__version__}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-isystem{d}" for d in cpp_extension.include_paths()),
           f"-isystem{sysconfig.get_paths()['include']}", "-isystem/opt/rocm/include",
           os.path.join(CSRC, "binding.cpp"), f"-L{libs}", "-ltorch_python", "-ltorch_cpu",
           "-lc10", "-lc10_hip", f"-Wl,-rpath,{libs}", "-o", NATIVE + ".tmp"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building the binding failed:\n{r.stderr}")
    os.replace(NATIVE + ".tmp", NATIVE)
    return NATIVE


def build(verbose: bool = False) -> str:
    out_dir = os.path.join(HERE, "_build")
    os.makedirs(out_dir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(out_dir, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
        if verbose and r.stderr:
            print(r.stderr)
        return obj

    with cf.ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        native = ex.submit(build_native)
        objs = list(ex.map(compile_one, SOURCES))
        try:
            native.result()
        except (ImportError, OSError, RuntimeError) as e:
            # the library does not depend on it: calls then go through ctypes,
            # but not through a file that was built from other sources
            if os.path.exists(NATIVE):
                os.remove(NATIVE)
            warnings.warn(f"{NATIVE} is not built: {e}", RuntimeWarning)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
