"""What the compiler reports about the built kernels' registers.  A kernel that keeps vector registers in memory waits for its own output
stores whenever it reads one back (loads and stores share one counter), which costs the rollout kernel up to 14 % of a ply."""
import os
import re
import struct
import subprocess

import pytest

import paper_2303_17503_amd as pg

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """(symbol, metadata text) of every kernel in the library: the notes of the AMD GPU code objects in it."""
    data = open(pg.LIB_PATH, "rb").read()
    out, at = [], 0
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:   # ELF64, little endian, ABI of the AMD GPU run time
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        part = tmp_path / f"code{at}.o"
        part.write_bytes(data[at: at + shoff + shentsize * shnum])
        notes = subprocess.run([READELF, "--notes", str(part)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n(?=  - )", notes.split("amdhsa.kernels:", 1)[1]):
            if m := re.search(r"\.symbol: +'?(\S+)\.kd", block):
                out.append((m.group(1), block))
        at += 64
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs ROCm's llvm-readelf")
def test_no_kernel_keeps_vector_registers_in_memory(tmp_path):
    found = kernels(tmp_path)
    names = " ".join(name for name, _ in found)
    for part in ("go_step_kernel", "go_step_superko_kernel", "go_rollout_kernel", "go_step_slots_kernel", "go_step_team_kernel", "go_rollout_team_kernel", "go_step_slots_team_kernel",
                 "go_step_superko_team_kernel", "hex_step_kernel", "hex_step_lane_kernel", "hex_rollout_kernel", "hex_rollout_lane_kernel", "hex_rollout_team_kernel"):
        assert part in names
    value = lambda block, key: int(re.search(rf"\.{key}: +(\d+)", block).group(1))  # noqa: E731
    spilled = {name: value(block, "vgpr_spill_count") for name, block in found if value(block, "vgpr_spill_count") or value(block, "private_segment_fixed_size")}
    assert not spilled, spilled
