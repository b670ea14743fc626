"""The strided geometry's longest messages (CPU only: a stand-in for hipLaunchKernel notes each launch's size and runs
nothing): a call is taken as far as the card's memory goes, in launches of fewer than 2^32 threads each."""
import os
import subprocess
import sys

import pytest

from paper_2506_17615_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = """
#include <hip/hip_runtime.h>
#include <stdint.h>
extern "C" { uint64_t g_most, g_launches; }
extern "C" hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    const uint64_t threads = (uint64_t)grid.x * block.x;
    if (threads > g_most) g_most = threads;
    ++g_launches;
    return hipSuccess;
}
"""
CHILD = """
import ctypes as C, os
from paper_2506_17615_amd import build
stub, lib = C.CDLL(os.environ["LD_PRELOAD"].split(":")[0]), C.CDLL(build.LIB_PATH)
most, launches = C.c_uint64.in_dll(stub, "g_most"), C.c_uint64.in_dll(stub, "g_launches")
lib.equarx_variant_workspace_bytes.restype = C.c_size_t
P, chunks = 3, 64
part, out, work = 1 << 20, 1 << 44, 1 << 45            # addresses that nothing touches
tab, null = (C.c_void_p * P)(*[part] * P), C.c_void_p(None)
for minishards in ((1 << 19) + 16, (1 << 20) - 1, (1 << 20) + 16, (1 << 20) + 80):      # up to 2^36 elements and a few more
    n = C.c_int64(1024 * chunks * minishards)
    for flags, count in ((0, 3), (8, 3), (1, 2), (9, 2)):
        most.value = launches.value = 0
        size = C.c_size_t(lib.equarx_variant_workspace_bytes(flags & ~8, P, n, chunks))
        got = lib.equarx_reduce_variant_hops_strided(tab, P, n, chunks, flags, C.c_void_p(out), C.c_void_p(work), size, null)
        assert (got, launches.value) == (0, count) and most.value < 1 << 32, (minishards, flags, got, launches.value, most.value)
print("ALL TAKEN")
"""


def test_the_longest_strided_messages_are_taken(tmp_path):
    src, stub = tmp_path / "launch.cpp", str(tmp_path / "liblaunch.so")
    src.write_text(STUB)
    include = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if not os.path.exists(os.path.join(include, "hip", "hip_runtime.h")):
        pytest.skip("the HIP headers are not installed here")
    subprocess.run(["g++", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", include, str(src), "-o", stub], check=True)
    build.ensure_built()
    env = dict(os.environ, PYTHONPATH=ROOT)
    env["LD_PRELOAD"] = stub + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    run = subprocess.run([sys.executable, "-c", CHILD], env=env, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "ALL TAKEN" in run.stdout, run.stdout[-2000:] + run.stderr[-2000:]
