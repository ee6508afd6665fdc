"""When a host output may be written through its mapping: only if the whole of
it lies in one pinned range.  The decision alone, compiled from the runtime's
header and run on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "alb_host.h"
int main(int, char **v) {
  auto x = [&](int i) { return std::strtoull(v[i], nullptr, 0); };
  std::printf("%d", (int)alb::range_holds((void *)x(1), x(2), (void *)x(3), x(4)));
  return 0;
}
"""
TOP = (1 << 64) - 1


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("range")
    (d / "r.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_1911_09135_amd", "csrc"), str(d / "r.cpp"), "-o",
                           str(d / "r")])
    return str(d / "r")


@pytest.mark.parametrize("base,size,p,nbytes,holds", [
    (0x10000, 4000, 0x10000, 4000, 1),      # the whole block
    (0x10000, 4000, 0x10000, 4004, 0),      # a block too short by one element
    (0x10000, 4096, 0x10000, 8192, 0),      # only the first page is pinned
    (0x10000, 4000, 0x10000 + 400, 3600, 1),  # a view to the block's end
    (0x10000, 4000, 0x10000 + 400, 3604, 0),
    (0x10000, 4000, 0x10000 + 4000, 0, 1),
    (0x10000, 4000, 0x10000 + 4000, 4, 0),
    (0x10000, 4000, 0x10000 + 4004, 0, 0),
    (0x10000, 4000, 0x10000 - 4, 8, 0),     # begins before it
    (0x10000, 0, 0x10000, 4, 0),
    (0x10000, 4000, 0x10000 + 8, TOP, 0),   # lengths that wrap
    (TOP - 4095, 4096, TOP - 4095, 4096, 1),
])
def test_range_holds(program, base, size, p, nbytes, holds):
    out = subprocess.check_output([program] + [str(x) for x in (base, size, p, nbytes)], text=True)
    assert int(out) == holds
