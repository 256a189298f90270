"""Builds libdodo.so (HIP, gfx950 only) and the binding's native calls (_dodo_torch.so) in-tree next to this file."""
from __future__ import annotations

import concurrent.futures
import importlib.util
import os
import subprocess
import sys
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libdodo.so")
NATIVE = os.path.join(_HERE, "_dodo_torch.so")
OBJ_DIR = os.path.join(_ROOT, "_build")

# packed fp32 VALU ops are switched off for every device translation unit
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-I", os.path.join(_ROOT, "include"), "-I", CSRC]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _build_native() -> None:
    """The extension module of the binding: host code against torch's own headers and libraries."""
    torch_dir = importlib.util.find_spec("torch").submodule_search_locations[0]
    inc, libs = os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", "-I", os.path.join(_ROOT, "include"),
           "-I", inc, "-I", os.path.join(inc, "torch", "csrc", "api", "include"), "-I", "/opt/rocm/include",
           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "dodo_torch.cpp"), "-o", NATIVE, "-L", libs,
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for dodo_torch.cpp:\n{r.stdout}\n{r.stderr}")


def build(verbose: bool = False) -> str:
    """Compiles every .hip source for gfx950, links libdodo.so and builds the binding's extension module.  Always recompiles."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        native = ex.submit(_build_native)
        objs = list(ex.map(_compile, srcs))
        native.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources, and {NATIVE}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
