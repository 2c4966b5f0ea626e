"""Builds libdllava.so (gfx950) in-tree with hipcc: one object per source, compiled in parallel, then linked; and _calls.so, the
native half of the Python binding, with the host compiler and torch's headers.  The library needs neither: where the second
cannot be built, the build says why and the binding does without it."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB_DIR = os.path.join(PKG, "lib")
LIB = os.path.join(LIB_DIR, "libdllava.so")
CALLS_SRC = os.path.join(PKG, "native", "calls.cpp")
CALLS = os.path.join(PKG, "_calls.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function"]
# packed-fp32 instructions are disabled for all device code
HIP_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unknown-warning-option", "-Wno-option-ignored"]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.rsplit(".", 1)[0] + ".o")
    cmd = [HIPCC, *COMMON]
    if src.endswith(".hip"):
        cmd += HIP_FLAGS
    cmd += ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    noise = ("is not a recognized feature for this target",)
    for line in r.stderr.splitlines():
        if line.strip() and not any(n in line for n in noise):
            print(line, file=sys.stderr)
    return obj


def build_calls() -> str:
    """Builds _calls.so; returns what prevented it, or an empty string.  An older one does not stay beside a newer library."""
    try:
        import sysconfig

        import torch
        from torch.utils.cpp_extension import include_paths
        os.makedirs(OBJ, exist_ok=True)
        obj, fresh = os.path.join(OBJ, "calls.o"), os.path.join(OBJ, "calls.so")
        version = f"{torch.__version__} {torch.version.git_version}"
        compiler = os.environ.get("CXX", "g++")
        compile_ = [compiler, "-O2", "-std=c++17", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    f'-DDLLAVA_TORCH_VERSION="{version}"', "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"]]
        for p in include_paths():
            compile_ += ["-isystem", p]
        # torch's libraries are in the process when the binding loads this one, and the binding hands it the library's functions
        link = [compiler, "-shared", obj, "-o", fresh, "-L", os.path.join(os.path.dirname(torch.__file__), "lib"),
                "-lc10", "-ltorch_cpu", "-ltorch_python"]
        for cmd in ([*compile_, "-c", CALLS_SRC, "-o", obj], link):
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise OSError(f"{cmd[0]} failed on {CALLS_SRC}:\n{r.stdout}\n{r.stderr}")
        os.replace(fresh, CALLS)
        return ""
    except (OSError, ImportError) as e:
        if os.path.exists(CALLS):
            os.remove(CALLS)
        return str(e)


def build(verbose: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    os.makedirs(LIB_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(jobs, len(srcs) + 1)) as ex:
        calls = ex.submit(build_calls)
        objs = list(ex.map(_compile, srcs))
        calls = calls.result()
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if calls:
        print(f"{CALLS} was not built, calls will take their arguments through ctypes: {calls}", file=sys.stderr)
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources")
    return LIB


if __name__ == "__main__":
    build()
