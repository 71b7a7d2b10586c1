"""Builds libcollm_lora.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcollm_lora.so")
# the Python binding's argument marshalling (CPython extension), named after the interpreter it is built for
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["api.cpp", "planner.cpp", "kernels_bf16.hip", "kernels_decode.hip", "kernels_f32.hip", "kernels_adapter.hip"]
HEADERS = ["plan.h", "planner.h", "kernels.h", "bf16_device.h"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-mcode-object-version=5",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _stale(out: str, deps) -> bool:
    if not os.path.exists(out):
        return True
    t = os.path.getmtime(out)
    return any(os.path.getmtime(d) > t for d in deps)


def _run(cmd, verbose: bool = False) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + " ".join(cmd) + "\n" + out)
    if verbose and out.strip():
        print(out, flush=True)


def build_marshal(force: bool = False, verbose: bool = False) -> bool:
    """Builds the extension with the host compiler.  The binding works without it (every call then takes its ctypes route), so
    a missing compiler or missing Python headers are a warning; returns whether the file is there."""
    src = os.path.join(CSRC, "marshal.cpp")
    stale = _stale(MARSHAL, [src, os.path.join(ROOT, "include", "collm_lora.h")])
    if not force and not stale:
        return True
    tmp = MARSHAL + ".tmp.%d" % os.getpid()
    try:
        # (it links nothing: the binding hands it the entry points of the library it has loaded)
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include"),
              "-I", sysconfig.get_paths()["include"], src, "-o", tmp], verbose)
        os.replace(tmp, MARSHAL)
    except (OSError, RuntimeError) as e:
        warnings.warn("the binding's compiled marshalling was not built, calls take the slower ctypes route: %s" % e)
        if stale and os.path.exists(MARSHAL):
            os.remove(MARSHAL)  # (of another source than the library: not to be loaded beside it)
    return os.path.exists(MARSHAL)


def build(force: bool = False, verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hdrs = [os.path.join(CSRC, h) for h in HEADERS] + [os.path.join(ROOT, "include", "collm_lora.h")]
    jobs = []
    objs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(objdir, src + ".o")
        objs.append(o)
        if force or _stale(o, [s] + hdrs):
            lang = ["-x", "hip"]
            jobs.append([hipcc] + FLAGS + lang + ["-c", s, "-o", o])

    with ThreadPoolExecutor(max_workers=4) as ex:
        list(ex.map(lambda cmd: _run(cmd, verbose), jobs))
    if force or jobs or _stale(LIB, objs):
        tmp = LIB + ".tmp.%d" % os.getpid()
        _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs, verbose)
        os.replace(tmp, LIB)
    build_marshal(force, verbose)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
