"""Blocks of wave_common.hpp by themselves, in small programs of their own."""
import os
import re
import subprocess

import pytest

import paper_2303_17503_amd.build as build

CSRC = os.path.join(os.path.dirname(build.__file__), "csrc")
GROW = """
#include "wave_common.hpp"
using namespace pgxwave;
// floods that begin as the whole of their set (f0 = s%d, f1 = s%d), which nothing needs afterwards
extern "C" __global__ void grown(uint32_t* p) {
  const uint32_t s[2] = {p[threadIdx.x], p[threadIdx.x + 64]};
  uint32_t f0 = s[%d], f1 = s[%d];
  Halves d0, d1;
  grow_pair(f0, f1, s[0], s[1], d0, d1);
  p[threadIdx.x] = f0 ^ f1 ^ d0.a ^ d0.b ^ d1.a ^ d1.b;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("first,second", [(0, 1), (1, 0)])
def test_a_flood_does_not_share_its_set_s_register(first, second, tmp_path):
    """The block of assembly reads the sets again after it has written the floods.  Where a flood is its own set at the start, the compiler may
    hold both in one register unless it is told not to."""
    src, asm = tmp_path / "grow.hip", tmp_path / "grow.txt"
    src.write_text(GROW % (first, second, first, second))
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-device-only", "-O3", "-std=c++17", "-I", CSRC, "-S", "-o", str(asm), str(src)], check=True, capture_output=True)
    steps = re.findall(r"v_bitop3_b32 (v\d+), v\d+, (v\d+), v\d+ bitop3:0xc8", asm.read_text())
    assert len(steps) == 8
    assert not {flood for flood, _ in steps} & {among for _, among in steps}, steps
