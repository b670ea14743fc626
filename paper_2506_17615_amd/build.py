"""Builds libequarx.so (the C-ABI HIP library) for gfx950 with hipcc and the binding's extension _marshal with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
INCLUDE = os.path.join(_ROOT, "include")
LIB_PATH = os.path.join(_PKG, "libequarx.so")
SOURCES = [os.path.join(CSRC, "equarx_api.hip"), os.path.join(CSRC, "equarx_devtools.hip")]
HEADERS = [os.path.join(CSRC, name) for name in ("equarx_device.hpp", "equarx_strided.hpp", "equarx_launch.hpp", "equarx_passes.hpp",
                                                  "equarx_devtools_kernels.hpp")]
HEADERS += [os.path.join(INCLUDE, "equarx.h"), os.path.join(INCLUDE, "equarx_devtools.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    # every rounding is written out in the kernels: no implicit multiply-add fusion
    "-ffp-contract=off",
    # packed-fp32 instructions stay out of the generated code.  The feature belongs to the gfx950 pass, which
    # honours it (tests/test_build_flags.py looks at the device assembly); hipcc hands -Xclang options to its
    # x86 host pass as well, which answers each with a harmless "not a recognized feature for this target".
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the leading kernel arguments arrive in scalar registers with the wave (gfx950's kernarg preload, 14 dwords at
    # most) instead of through a scalar load that every kernel would begin by waiting for
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-shared", "-fPIC",
    "-I", INCLUDE, "-I", CSRC,
]

# the binding's native half: a Python extension against torch's headers, host code only.  It belongs to one interpreter
# and one torch, so its name carries the one and it knows the other; without it the binding marshals in Python.
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.cpp")
MARSHAL_PATH = os.path.join(_PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
MARSHAL_FLAGS = ["-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM"]


STAMP_PATH = LIB_PATH + ".stamp"
MARSHAL_STAMP_PATH = MARSHAL_PATH + ".stamp"


def source_digest() -> str:
    """SHA-256 over the build flags and the text of every source and header the library is built from."""
    import hashlib
    h = hashlib.sha256(" ".join(HIPCC_FLAGS[:-4]).encode())      # flags without the -I paths (machine-specific)
    for path in SOURCES + HEADERS:
        h.update(os.path.basename(path).encode())
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def _marshal_command() -> list:
    import torch
    home = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), *MARSHAL_FLAGS, f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DEQUARX_TORCH="{torch.__version__}"', "-I", sysconfig.get_paths()["include"], "-isystem",
            os.path.join(home, "include"), "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
            "-I", INCLUDE, MARSHAL_SOURCE, "-o", MARSHAL_PATH, "-L", os.path.join(home, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def _marshal_digest() -> str:
    import hashlib
    import torch
    h = hashlib.sha256(" ".join([*MARSHAL_FLAGS, str(torch._C._GLIBCXX_USE_CXX11_ABI), torch.__version__,
                                 str(sysconfig.get_config_var("SOABI"))]).encode())
    for path in (MARSHAL_SOURCE, os.path.join(INCLUDE, "equarx.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def _differs(path: str, stamp: str, digest: str) -> bool:
    if not os.path.exists(path) or not os.path.exists(stamp):
        return True
    with open(stamp) as f:
        return f.read().strip() != digest


def library_is_stale() -> bool:
    """True if the library is not there, or was not built from the sources as they are now.  Decided
    by content (a digest written next to the library at build time), not by file times, which a copy of the tree
    to another machine does not keep."""
    return _differs(LIB_PATH, STAMP_PATH, source_digest())


def extension_is_stale() -> bool:
    """The same for the binding's extension, with the interpreter and the torch it was built for.  Without torch there
    is no use for it."""
    try:
        digest = _marshal_digest()
    except ImportError:
        return False
    return _differs(MARSHAL_PATH, MARSHAL_STAMP_PATH, digest)


def is_stale() -> bool:
    return library_is_stale() or extension_is_stale()


def _build_library(verbose: bool) -> None:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *SOURCES, "-o", LIB_PATH]
    if verbose:
        print(" ".join(cmd), flush=True)
    digest = source_digest()
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + proc.stdout + proc.stderr)
    with open(STAMP_PATH, "w") as f:
        f.write(digest + "\n")


def _build_marshal() -> None:
    try:
        cmd, digest = _marshal_command(), _marshal_digest()
    except ImportError:         # a caller of the C interface needs no torch
        print("torch is not installed: the library is built without the binding's extension", flush=True)
        return
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("the binding's extension does not compile:\n" + proc.stdout + proc.stderr)
    with open(MARSHAL_STAMP_PATH, "w") as f:
        f.write(digest + "\n")


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile the library and the binding's extension, or with force=False what is stale of them; returns the library's
    path.  Raises if a compiler fails."""
    if force or library_is_stale():
        _build_library(verbose)
    if force or extension_is_stale():
        _build_marshal()
    return LIB_PATH


def ensure_built() -> str:
    """What tests, smoke and bench call before loading the library: build it if it is missing, and never run a
    library that is older than the sources beside it -- rebuild where hipcc exists, refuse where it does not."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if library_is_stale() and os.path.exists(LIB_PATH) and not os.path.exists(hipcc):
        raise RuntimeError(f"{LIB_PATH} is older than its sources and {hipcc} is not there to rebuild it")
    return build(force=False)


if __name__ == "__main__":
    print(build(verbose=True))
