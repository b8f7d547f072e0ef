"""Host code of the library on the CPU, compiled from its own sources, and the
benchmark's digest of them."""
import inspect
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_03318_amd", "csrc")
CLANGXX = "/opt/rocm/lib/llvm/bin/clang++"
INC = ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _run(exe):
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ALL OK" in r.stdout, (r.stdout[-2000:], r.stderr[-4000:])


def test_sizes_of_launches_and_arrays(tmp_path):
    """Chunks and tiles at 2^31 - 1 tasks (a sum in 32 bits wraps there), and
    room for every word of the removal strings that a lane reads."""
    if not os.path.exists(CLANGXX):
        pytest.skip("%s not present" % CLANGXX)
    exe = str(tmp_path / "layout")
    subprocess.check_call([CLANGXX, "-O1", "-std=c++17", *INC, os.path.join(ROOT, "tests", "host", "layout.cpp"),
                           "-o", exe])
    _run(exe)


def test_pinned_memory_of_ended_threads(tmp_path):
    """Host threads that come and go share their pinned buffers, and
    dd_release_cache returns them (the API layer alone, on host memory)."""
    hipcc = "/opt/rocm/bin/hipcc"
    if not (os.path.exists(CLANGXX) and os.path.exists(hipcc)):
        pytest.skip("no ROCm compilers")
    obj, exe = str(tmp_path / "dd_api.o"), str(tmp_path / "pinned")
    subprocess.check_call([hipcc, "--offload-host-only", "-O1", "-std=c++17", *INC[2:], "-c",
                           os.path.join(CSRC, "dd_api.hip"), "-o", obj], stderr=subprocess.DEVNULL)
    subprocess.check_call([CLANGXX, "-O1", "-std=c++17", *INC, os.path.join(ROOT, "tests", "host", "pinned.cpp"), obj,
                           "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-pthread", "-o", exe])
    _run(exe)


def test_schedule_without_memory_for_every_record(tmp_path):
    """dd_levelize succeeds where all but the records of the one-variant
    kernel fit (host code alone: launches do nothing, allocations past a
    limit fail)."""
    hipcc = "/opt/rocm/bin/hipcc"
    if not (os.path.exists(CLANGXX) and os.path.exists(hipcc)):
        pytest.skip("no ROCm compilers")
    obj, exe = str(tmp_path / "k_levelize.o"), str(tmp_path / "levelize_memory")
    subprocess.check_call([hipcc, "--offload-host-only", "-O1", "-std=c++17", *INC[2:], "-c",
                           os.path.join(CSRC, "k_levelize.hip"), "-o", obj], stderr=subprocess.DEVNULL)
    subprocess.check_call([CLANGXX, "-O1", "-std=c++17", *INC, os.path.join(ROOT, "tests", "host", "levelize_memory.cpp"),
                           obj, "-pthread", "-Wl,--unresolved-symbols=ignore-all", "-o", exe])   # (no device code)
    _run(exe)


def test_digest_covers_the_sources_of_the_kernel():
    """bench.py quotes a measured traffic only for the sources it was measured
    on: every file that the kernel includes counts."""
    import bench
    named = set(re.findall(r"csrc/([\w.]+)", inspect.getsource(bench.kernel_source_digest)))
    todo, seen = ["k_simulate.hip"], set()
    while todo:
        f = todo.pop()
        seen.add(f)
        with open(os.path.join(CSRC, f)) as fh:
            inc = re.findall(r'#include "([\w.]+)"', fh.read())
        todo += [i for i in inc if i not in seen and os.path.exists(os.path.join(CSRC, i))]
    assert seen <= named, seen - named
