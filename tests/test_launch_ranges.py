"""Launches that grow with the batch are cut below HIP's 2^32 threads (compiled
for the host): every item once, in order, each range within the limit."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11709_amd", "csrc")

PROGRAM = r"""
#include "xrd_internal.h"
#include <stdio.h>
#include <stdlib.h>
int main(int, char **v) {
  xrd::launch_ranges(atoll(v[1]), atoll(v[2]), [](int64_t f, int64_t n) { printf("%lld %lld\n", (long long)f, (long long)n); });
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the HIP headers not available")
    d = tmp_path_factory.mktemp("ranges")
    (d / "m.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", "-I", CSRC,
                           str(d / "m.cpp"), "-o", str(d / "m")])
    return str(d / "m")


# items and threads of each: grids of 16384 points (128 points to 256 threads)
# on either side of the limit, chunks of 1024 threads, one item near it
@pytest.mark.parametrize("n,threads", [(0, 256), (1, 2 ** 32 - 1), (131071, 32768), (131072, 32768), (600000, 16384),
                                       (2 ** 22 - 1, 1024), (2 ** 22, 1024), (2 ** 24, 1024), (3, 2 ** 31)])
def test_ranges(exe, n, threads):
    out = subprocess.run([exe, str(n), str(threads)], capture_output=True, text=True, check=True).stdout
    at = 0
    for first, count in (map(int, line.split()) for line in out.splitlines()):
        assert first == at and count > 0 and count * threads < 2 ** 32
        at += count
    assert at == n
    if n * threads < 2 ** 32:
        assert len(out.splitlines()) == (n > 0)
