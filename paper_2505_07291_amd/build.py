"""Builds libgrpo.so (the C-ABI library with the gfx950 HIP kernels) and the binding's native part in-tree."""
from __future__ import annotations

import concurrent.futures
import glob
import hashlib
import os
import shutil
import subprocess

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
SOURCES = [os.path.join(_PKG, "csrc", "grpo.hip")]
INCLUDE = os.path.join(_ROOT, "include")
LIB_PATH = os.path.join(_PKG, "libgrpo.so")
FASTCALL_SOURCE = os.path.join(_PKG, "csrc", "fastcall.cpp")

# -packed-fp32-ops is switched off on purpose: packed fp32 forms generated from plain
# float code have produced wrong results on the test machines.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# the parts of grpo.hip, compiled at the same time
PARTS = [["-DGRPO_ROWS_APART"]] + [["-DGRPO_ROWS_OF=%s, %s" % (dt, aux)] for dt in ("GRPO_BF16", "GRPO_F32") for aux in ("false", "true")]


def find_hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: libgrpo needs the ROCm compiler to build")


def build_library(verbose: bool = False) -> str:
    """Compiles the library unconditionally and returns its path."""
    tmp = LIB_PATH + ".tmp.%d" % os.getpid()
    objects = ["%s.%d.o" % (tmp, i) for i in range(len(PARTS))]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        return subprocess.run(cmd, capture_output=True, text=True)

    base = [find_hipcc()] + HIPCC_FLAGS
    try:
        with concurrent.futures.ThreadPoolExecutor(len(PARTS)) as pool:
            results = list(pool.map(lambda part: run(base + part[0] + ["-I", INCLUDE, "-c", "-o", part[1]] + SOURCES),
                                    zip(PARTS, objects)))
        results.append(run(base + ["-shared", "-o", tmp] + objects) if all(r.returncode == 0 for r in results) else results[0])
        for res in results:
            if res.returncode != 0:
                raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    finally:
        for path in objects:
            if os.path.exists(path):
                os.unlink(path)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


def compile_fastcall(source: str, out: str, verbose: bool = False) -> None:
    """Compiles host code against torch's headers into a Python extension."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = out + ".tmp.%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM"]
    for path in (os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                 sysconfig.get_paths()["include"], "/opt/rocm/include"):
        cmd += ["-isystem", path]
    cmd += ["-I", INCLUDE, "-o", tmp, source, "-L" + os.path.join(root, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout + res.stderr)
    os.replace(tmp, out)


def fastcall_path() -> str:
    """Where the binding's native part lies.  The library's argument types, the order of its own arguments and torch's C++
    interface are compiled into it, so its name says which sources, which torch and which Python it was built for:
    one that was left over from others has another name and is never loaded."""
    import sysconfig
    import torch
    tag = hashlib.sha256(repr((torch.__version__, torch.version.git_version, sysconfig.get_config_var("SOABI"))).encode())
    for path in (os.path.join(INCLUDE, "grpo.h"), FASTCALL_SOURCE):
        with open(path, "rb") as f:
            tag.update(f.read())
    return os.path.join(_PKG, "_fastcall.%s.so" % tag.hexdigest()[:16])


def build_fastcall(verbose: bool = False) -> str:
    """Compiles the binding's native part, removes those of other sources, and returns its path."""
    path = fastcall_path()
    compile_fastcall(FASTCALL_SOURCE, path, verbose)
    for old in glob.glob(os.path.join(_PKG, "_fastcall*.so")):
        if old != path:
            try:
                os.unlink(old)
            except FileNotFoundError:  # another process has built at the same time
                pass
    return path


def is_stale() -> bool:
    if not os.path.exists(LIB_PATH) or not os.path.exists(fastcall_path()):
        return True
    t = os.path.getmtime(LIB_PATH)
    deps = SOURCES + [os.path.join(_PKG, "csrc", f) for f in ("lmhead.hpp", "lm_plan.hpp")] + [os.path.join(INCLUDE, "grpo.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_fastcall(verbose=True))
