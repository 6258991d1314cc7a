"""Wait states that the hardware leaves to software, in the built gfx950 code.

The compiler's hazard pass does not look inside assembly strings, so the LDS
DMAs written there have to bring their own: one wait state between a scalar
write of M0 and a load into LDS, which takes its LDS address from M0.
Shown on the disassembly of the library that was built here."""

import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_2601_21622_amd as sd
from paper_2601_21622_amd import build as sd_build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

M0_WAIT = 1


def to_lds(op, args):
    return op.startswith(("global_load_lds", "buffer_load", "scratch_load_lds")) and (
        "_lds" in op or re.search(r"\blds\b", args) is not None)


def find_hazards(lines):
    """(line, why) of every instruction that follows another too closely, in
    straight-line order; a wait state is an instruction, s_nop n is n + 1."""
    found, loads, m0_at, now = [], 0, None, 0
    for line in lines:
        text = line.split("//")[0].split(";")[0].strip()
        if not text or text.endswith(":"):
            continue
        op, _, args = text.partition(" ")
        if to_lds(op, args):
            loads += 1
            if m0_at is not None and now - m0_at < M0_WAIT:
                found.append((text, "M0"))
        now += int(args, 0) + 1 if op == "s_nop" else 1
        if op.startswith("s_") and re.match(r"m0\b", args.strip()):
            m0_at = now
    return found, loads


def test_the_scan_sees_a_hazard():
    bad = ["\ts_mov_b32 m0, s4", "\tglobal_load_lds_dwordx4 v[2:3], off nt"]
    assert len(find_hazards(bad)[0]) == 1
    assert find_hazards([bad[0], "\ts_nop 0", bad[1]]) == ([], 1)
    assert find_hazards([bad[0], "\tv_mov_b32_e32 v1, 0", bad[1]]) == ([], 1)
    assert len(find_hazards(["\ts_add_i32 m0, s3, 0x400", "\tbuffer_load_dwordx4 v2, s[0:3], 0 offen lds"])[0]) == 1
    assert find_hazards(["\ts_mov_b32 m0, s3", "\tbuffer_load_dwordx4 v2, s[0:3], 0 offen"]) == ([], 0)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_built_code_has_no_hazard(tmp_path):
    sd.library()
    lib = str(tmp_path / "lib.so")
    shutil.copy(sd_build.LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    objects = glob.glob(lib + ".*gfx950*")
    assert len(objects) >= len(sd_build.SOURCES) - 1
    total = 0
    for o in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", o], check=True, capture_output=True, text=True).stdout
        found, loads = find_hazards(text.splitlines())
        total += loads
        assert not found, f"{os.path.basename(o)}: {len(found)}, first {found[:3]}"
    assert total > 1000  # the attention's and the projection's DMAs were among them
