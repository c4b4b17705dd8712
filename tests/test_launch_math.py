"""Index and plan arithmetic of the launches (csrc/launch_math.h), compiled with the host compiler and checked at sizes
that no GPU test launches."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "launch_math.h"
extern "C" {
unsigned clear_blocks() { return fv::kClearBlocks; }
unsigned clear_threads() { return fv::kClearThreads; }
int clears(unsigned block) { return fv::clears_counters(block); }
void share(unsigned block, unsigned thread, unsigned blocks, int* out) {
    const fv::CounterShare s = fv::counter_share(block, thread, blocks);
    out[0] = s.first;
    out[1] = s.step;
}
}
"""


@pytest.fixture(scope="module")
def math(tmp_path_factory):
    cxx = shutil.which("g++") or "/opt/rocm/bin/amdclang++"
    d = tmp_path_factory.mktemp("launch_math")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2503_23367_amd", "csrc"), "-o", str(so), str(src)], check=True)
    return C.CDLL(str(so))


def _share(math, block, thread, blocks):
    out = (C.c_int * 2)()
    math.share(C.c_uint(block), C.c_uint(thread), C.c_uint(blocks), out)
    return out[0], out[1]


@pytest.mark.parametrize("blocks", [1, 2, 255, 256, 257, 1 << 23, (1 << 23) + 1, 1 << 24, (1 << 31) - 1])
def test_counter_shares_stay_in_range_and_cover_every_counter_once(math, blocks):
    """A flat index over all workgroups passes 2^31 at 2^23 workgroups of 256 threads, turns negative, and a thread of a
    launch without any counters then stores through the null pointer."""
    threads, most = math.clear_threads(), math.clear_blocks()
    for block in {0, 1, most - 1, most, min(blocks, 1 << 23), (1 << 23) - 1, (1 << 23) + 5, blocks - 1}:
        if not 0 <= block < blocks or not math.clears(C.c_uint(block)):
            continue
        for thread in (0, 1, threads - 1):
            first, step = _share(math, block, thread, blocks)
            assert 0 <= first < step <= most * threads, (block, thread)
    for n in (0, 1, 300, 70000):
        seen = [0] * n
        for block in range(min(blocks, most + 2)):
            if math.clears(C.c_uint(block)):
                for thread in range(threads):
                    first, step = _share(math, block, thread, blocks)
                    for i in range(first, n, step):
                        seen[i] += 1
                    if first >= n:
                        break
        assert seen == [1] * n
