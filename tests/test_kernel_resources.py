"""Registers of the reduction kernels as built: they decide how many waves a SIMD holds."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_17694_amd.binding import LIB_PATH

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def resources(folder):
    """Mangled kernel name -> (vector registers, bytes of scratch memory of a lane)"""
    if not os.path.exists(OBJDUMP) or not os.path.exists(READELF):
        pytest.skip("llvm-objdump or llvm-readelf is not installed")
    shutil.copy(LIB_PATH, folder / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=folder, check=True, capture_output=True)
    (image,) = [f for f in os.listdir(folder) if "gfx950" in f]
    notes = subprocess.run([READELF, "--notes", image], cwd=folder, check=True, capture_output=True, text=True).stdout
    out = {}
    for block in re.split(r"\n  - (?=\.)", notes):
        name = re.search(r"\.name:\s+(_Z\S+)", block)
        if name:
            out[name.group(1)] = tuple(int(re.search(rf"\.{k}:\s+(\d+)", block).group(1))
                                       for k in ("vgpr_count", "private_segment_fixed_size"))
    return out


def waves_per_simd(registers):
    return 512 // (-(-registers // 8) * 8)          # 512 per lane, handed out in eights


def test_reductions_of_long_lists_leave_room_for_as_many_waves(tmp_path):
    """A large launch in which a few lists are long and most short is bound by the waves of a CU: its kernel (form 2) must
    not keep the rows of two chunks at once.  Four waves fit, as with one kernel for lists of every length; none spills."""
    seen = {}
    for name, (registers, scratch) in resources(tmp_path).items():
        m = re.search(r"merge_kernelILi(\d)ELi(\d+)ELi(\d)ELi(\d)E", name)
        if m:
            assert scratch == 0, name
            seen[tuple(int(x) for x in m.groups())] = registers
    assert len(seen) == 2 * 5 * 3                   # two data types, five sizes of row groups, three forms
    for (dtype, d, rows, form), registers in seen.items():
        assert waves_per_simd(registers) >= (5 if form == 0 else 4), (dtype, d, rows, form, registers)
        if form == 2:
            assert registers <= seen[dtype, d, rows, 1], (dtype, d, rows, registers)
