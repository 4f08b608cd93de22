"""Checks of the library's own device code (disassembled from the build)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2302_07594_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def shifts_at_the_end_of_the_registers(listing):
    """(kernel, instruction) of every 64-bit shift whose amount is a VGPR that
    ends a block of eight and is followed by none that the kernel uses: such a
    register may be the last one allocated, and the shift then takes its
    amount from v0. The compiler moves it on gfx90a only."""
    found, kernel, used, shifts = [], None, set(), []

    def close():
        found.extend((kernel, text) for text, n in shifts if n % 8 == 7 and n + 1 not in used)

    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.+)>:", line)
        if head:
            close()
            kernel, used, shifts = head.group(1), set(), []
            continue
        text = line.split("//")[0].strip()
        for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
            used.update(range(int(lo), int(hi) + 1))
        used.update(int(n) for n in re.findall(r"\bv(\d+)\b", text))
        shift = re.match(r"v_(?:lshl|lshr|ashr)rev_[bi]64\S*\s+v\[\d+:\d+\],\s*v(\d+)\b", text)
        if shift:
            shifts.append((text, int(shift.group(1))))
    close()
    return found


def test_shift_scan_on_a_listing():
    text = """
0000 <bad>:
	v_lshrrev_b64 v[74:75], v95, v[56:57]    // 0000: D290004A
	v_mov_b32_e32 v94, v3                    // 0008: 7E00
0010 <next_register_used>:
	v_lshlrev_b64 v[2:3], v7, v[4:5]
	v_mov_b32_e32 v8, 0
0020 <inside_a_block>:
	v_ashrrev_i64 v[2:3], v6, v[4:5]
0030 <scalar_amount>:
	v_ashrrev_i64 v[6:7], s7, v[4:5]
"""
    assert shifts_at_the_end_of_the_registers(text) == [
        ("bad", "v_lshrrev_b64 v[74:75], v95, v[56:57]")]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_64_bit_shift_takes_its_amount_from_the_last_register(tmp_path):
    shutil.copyfile(build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True,
                   capture_output=True)
    objects = glob.glob(str(tmp_path / "lib.so*gfx950*"))
    assert len(objects) >= 8
    kernels = 0
    for obj in objects:
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True,
                                 capture_output=True, text=True).stdout
        kernels += listing.count(">:\n")
        found = shifts_at_the_end_of_the_registers(listing)
        assert not found, "\n".join(f"{k}: {t}" for k, t in found)
    assert kernels > 50
