"""Builds the HIP library (``libemb_hip.so``) for gfx950 with hipcc, and with g++ the CPython module
(``_calls.*.so``) that marshals the shortest calls.

The library is plain C ABI (``include/emb.h``): one ``hipcc -shared`` line.  The module knows torch tensors (it is
compiled against the layout of those of one torch, which its file's name says) and is of use to ``binding.py`` only,
which does without it where it is missing.
"""
from __future__ import annotations

import contextlib
import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libemb_hip.so")

CALLS_SRC = os.path.join(CSRC, "calls.cpp")

CXX = os.environ.get("CXX", "g++")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 instructions are switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(ROOT, "include", "emb.h")]
    return os.path.getmtime(LIB) < max(os.path.getmtime(d) for d in deps)


def calls_path() -> str:
    """The module for this interpreter and this torch: those of others have other names."""
    import re
    import sysconfig

    import torch
    return os.path.join(PKG, "_calls.%s-torch-%s.so" % (sysconfig.get_config_var("SOABI"),
                                                        re.sub(r"[^A-Za-z0-9.+]", "_", torch.__version__)))


def _calls_failed_path() -> str:
    """Empty file left by an attempt to compile the module that failed."""
    return os.path.join(PKG, "_build", os.path.basename(calls_path()) + ".failed")


def _older_than_calls_sources(path: str) -> bool:
    deps = (CALLS_SRC, os.path.join(ROOT, "include", "emb.h"))
    return not os.path.exists(path) or os.path.getmtime(path) < max(os.path.getmtime(d) for d in deps)


def calls_is_stale() -> bool:
    return _older_than_calls_sources(calls_path())


def calls_can_be_built() -> bool:
    """False where the file cannot be written, and after a failed attempt until the sources change."""
    return os.access(PKG, os.W_OK) and _older_than_calls_sources(_calls_failed_path())


def build_calls(verbose: bool = True) -> str:
    """Compile ``csrc/calls.cpp`` against the torch that is installed."""
    import sysconfig

    import torch
    t, out, failed = os.path.dirname(torch.__file__), calls_path(), _calls_failed_path()
    part = out + ".%d" % os.getpid()
    try:
        _run([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
              "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(t, "include"),
              "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
              CALLS_SRC, "-o", part, "-L", os.path.join(t, "lib"), "-ltorch_python", "-lc10"], verbose)
    except (OSError, RuntimeError):
        os.makedirs(os.path.dirname(failed), exist_ok=True)
        with open(failed, "w"):
            pass
        raise
    os.replace(part, out)   # other processes see all of it or none
    with contextlib.suppress(FileNotFoundError):
        os.remove(failed)
    return out


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the device-only target feature and says so: harmless
    log = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if log.strip() and verbose:
        print(log, flush=True)
    if p.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + log)


def build(verbose: bool = True, jobs: int = 6) -> str:
    """Compile every ``csrc/*.hip`` for gfx950 (in parallel) and link ``libemb_hip.so``; then the module of ``csrc/calls.cpp``,
    whose failure is reported and no error."""
    from concurrent.futures import ThreadPoolExecutor

    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    compile_flags = [f for f in FLAGS if f != "-shared"]
    objs = []
    cmds = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        cmds.append([HIPCC, *compile_flags, *inc, "-c", src, "-o", obj])
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(cmds)))) as ex:
        list(ex.map(lambda c: _run(c, verbose), cmds))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], verbose)
    try:
        build_calls(verbose)
    except (OSError, RuntimeError) as e:
        print("no module of csrc/calls.cpp, calls go through ctypes: %s" % e, file=sys.stderr, flush=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
