"""Builds libfc.so (HIP kernels + C ABI) for gfx950 with hipcc, in tree.

    python -m paper_2407_13585_amd.build [--force]

hipcc cross-compiles without a GPU.  Floating-point contraction is off for
device and host code so that a*x+b is two roundings everywhere (element
functions must be bit-exact across fused and unfused execution).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfc.so")
# the call of a bound program as a Python type (csrc/bound.c); the name says which interpreter it was compiled for
BOUND = os.path.join(HERE, "_bound_call" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["api.hip", "run.hip", "instances.hip", "interp.hip", "generic_folds.hip", "generic_rows.hip", "generic_scans.hip", "model.cpp",
           "plan.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-Wall", "-Wno-unused-function"]
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _headers():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hpp", ".h"))]
    hs.append(os.path.join(os.path.dirname(HERE), "include", "fc.h"))
    return hs


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src, force):
    obj = os.path.join(OBJ, src + ".o")
    path = os.path.join(CSRC, src)
    if not force and not _stale(obj, [path] + _headers()):
        return obj, ""
    cmd = [HIPCC] + COMMON
    if src.endswith(".hip"):
        cmd += DEVICE
    cmd += ["-c", path, "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError(f"{' '.join(cmd)}\n{p.stdout}\n{p.stderr}")
    return obj, p.stderr


def build_bound(force: bool = False) -> str:
    """The extension module that binding.BoundRun is made on: host code only, against this interpreter's headers."""
    src = os.path.join(CSRC, "bound.c")
    if force or _stale(BOUND, [src]):
        cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], src,
               "-o", BOUND + f".{os.getpid()}"]
        p = subprocess.run(cmd, capture_output=True, text=True)
        if p.returncode != 0:
            raise RuntimeError(f"{' '.join(cmd)}\n{p.stdout}\n{p.stderr}")
        os.replace(BOUND + f".{os.getpid()}", BOUND)
    return BOUND


def build(force: bool = False, verbose: bool = False) -> str:
    try:
        build_bound(force)
    except (OSError, RuntimeError) as e:               # no compiler, no headers of this interpreter: binding.py does without
        print(f"not built: {e}", file=sys.stderr)
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        results = list(ex.map(lambda s: _compile(s, force), SOURCES))
    objs = [o for o, _ in results]
    if verbose:
        for _, log in results:
            if log.strip():
                print(log, file=sys.stderr)
    if force or _stale(LIB, objs):
        cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
        p = subprocess.run(cmd, capture_output=True, text=True)
        if p.returncode != 0:
            raise RuntimeError(f"{' '.join(cmd)}\n{p.stdout}\n{p.stderr}")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
