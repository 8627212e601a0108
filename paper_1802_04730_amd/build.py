"""Build libtc355.so (hipcc, gfx950) and the binding's native calls _fast.so (g++) in-tree."""
from __future__ import annotations

import glob
import hashlib
import os
import subprocess
import sys
import sysconfig
import threading
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtc355.so")
STAMP = LIB + ".srchash"  # hash of the sources the library was built from
FAST = os.path.join(HERE, "_fast.so")  # the binding's calls in native code
FAST_SOURCE = os.path.join(CSRC, "fast_call.cpp")
FAST_STAMP = FAST + ".srchash"
FAST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _deps():
    return sorted(glob.glob(os.path.join(CSRC, "*.h*"))) + [os.path.join(HERE, "..", "include", "tc355.h")]


def source_hash() -> str:
    """Hash of everything the library is compiled from (file contents, not time stamps: a copy of the tree keeps it)."""
    h = hashlib.sha256(" ".join(HIPCC_FLAGS).encode())
    for d in _deps():
        h.update(os.path.basename(d).encode())
        with open(d, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def is_stale() -> bool:
    """True if there is no built library or it was built from other sources than the tree holds now."""
    if not os.path.exists(LIB) or not os.path.exists(STAMP):
        return True
    with open(STAMP) as f:
        return f.read().strip() != source_hash()


def hipcc_path() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def have_hipcc() -> bool:
    return os.access(hipcc_path(), os.X_OK)


def fast_hash() -> str:
    """Hash of what _fast.so is compiled from: its source, the flags, and the interpreter and torch whose headers it uses."""
    import torch

    h = hashlib.sha256(("%s %s %s" % (sys.version, torch.__version__, " ".join(FAST_FLAGS))).encode())
    with open(FAST_SOURCE, "rb") as f:
        h.update(f.read())
    return h.hexdigest()


def fast_is_stale() -> bool:
    if not os.path.exists(FAST) or not os.path.exists(FAST_STAMP):
        return True
    with open(FAST_STAMP) as f:
        return f.read().strip() != fast_hash()


def _compile(cmd: list, out: str, compiler: str, verbose: bool) -> str:
    """Run a compiler line that ends before its output's name and write `out` as a whole: another process may be loading it, or
    making it too.  Returns what the compiler said."""
    if verbose:
        print(" ".join(cmd + ["-o", out]), flush=True)
    part = "%s.%d.%d.part" % (out, os.getpid(), threading.get_ident())
    try:
        r = subprocess.run(cmd + ["-o", part], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(compiler + " failed:\n" + r.stdout + r.stderr)
        os.replace(part, out)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return r.stderr


def torch_module_command(source: str) -> list:
    """g++ line, but for the output's name, of a Python module that uses torch's headers."""
    import torch

    t = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(hipcc_path()))
    return [os.environ.get("CXX", "g++")] + FAST_FLAGS + [
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
            "-I" + os.path.join(t, "include"), "-I" + os.path.join(t, "include", "torch", "csrc", "api", "include"),
            "-I" + os.path.join(rocm, "include"), "-I" + sysconfig.get_paths()["include"], source,
            "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build_fast(verbose: bool = False) -> str:
    """Compile the binding's native calls against torch's headers; returns the module's path."""
    made_from = fast_hash()  # (of the source as the compiler finds it)
    _compile(torch_module_command(FAST_SOURCE), FAST, "g++", verbose)
    with open(FAST_STAMP, "w") as f:
        f.write(made_from + "\n")
    return FAST


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every HIP source into libtc355.so, and _fast.so; returns the library path.

    _fast.so only saves host time: where it cannot be built, that is a warning."""
    if force or is_stale():
        made_from = source_hash()  # (of the sources as the compiler finds them)
        said = _compile([hipcc_path()] + HIPCC_FLAGS + sources(), LIB, "hipcc", verbose)
        with open(STAMP, "w") as f:
            f.write(made_from + "\n")
        if verbose:
            noise = "is not a recognized feature for this target"
            for line in said.splitlines():
                if noise not in line:
                    print(line)
    if force or fast_is_stale():
        try:
            build_fast(verbose)
        except (RuntimeError, OSError) as e:
            warnings.warn("_fast.so could not be built: calls go through ctypes, some microseconds slower (%s)" % e, RuntimeWarning, stacklevel=2)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
