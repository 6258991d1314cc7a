"""Wait states that the hardware leaves to software, in the built gfx950 code.

The compiler's hazard pass does not look inside assembly strings, so the LDS
DMAs written there have to bring their own: one wait state between a scalar
write of M0 and a load into LDS, which takes its LDS address from M0, and five
between a vector instruction's write of a scalar register (readfirstlane) and
a memory instruction that reads it.  Shown on the disassembly of the library
that was built here."""

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
SGPR_WAIT = 5


def to_lds(op, args):
    return op.startswith(("global_load_lds", "buffer_load", "scratch_load_lds")) and (
        "_lds" in op or re.search(r"\blds\b", args) is not None)


def scalars(arg):
    """Numbers of the scalar registers an operand names."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", arg)
    if m is None:
        return range(0)
    return range(int(m[3]), int(m[3]) + 1) if m[3] else range(int(m[1]), int(m[2]) + 1)


def find_hazards(lines):
    """(line, why) of every instruction that follows another too closely, in
    straight-line order; a wait state is an instruction, s_nop n is n + 1."""
    found, loads, m0_at, now = [], 0, None, 0
    vector_at = {}  # scalar register -> when a vector instruction wrote it
    for line in lines:
        text = line.split("//")[0].split(";")[0].strip()
        if not text or text.endswith(":"):
            continue
        op, _, args = text.partition(" ")
        if to_lds(op, args):
            loads += 1
            if m0_at is not None and now - m0_at < M0_WAIT:
                found.append((text, "M0"))
        words = re.split(r",\s*|\s+", args.strip())
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            if any(now - vector_at.get(r, -SGPR_WAIT) < SGPR_WAIT for w in words for r in scalars(w)):
                found.append((text, "scalar register"))
        now += int(args, 0) + 1 if op == "s_nop" else 1
        if op.startswith("s_") and re.match(r"m0\b", args.strip()):
            m0_at = now
        if op.startswith("v_"):  # the destination, and a second one (carry out, scale)
            for w in words[:2] if re.search(r"_co_|div_scale|mad_[iu]64", op) else words[:1]:
                vector_at.update((r, now) for r in scalars(w))
        elif op.startswith("s_"):
            for r in scalars(words[0]):
                vector_at.pop(r, None)
    return found, loads


def test_the_scan_sees_a_hazard():
    bad = ["\ts_mov_b32 m0, s4", "\tglobal_load_lds_dwordx4 v[2:3], off nt"]
    assert len(find_hazards(bad)[0]) == 1
    assert find_hazards([bad[0], "\ts_nop 0", bad[1]]) == ([], 1)
    assert find_hazards([bad[0], "\tv_mov_b32_e32 v1, 0", bad[1]]) == ([], 1)
    assert len(find_hazards(["\ts_add_i32 m0, s3, 0x400", "\tbuffer_load_dwordx4 v2, s[0:3], 0 offen lds"])[0]) == 1
    assert find_hazards(["\ts_mov_b32 m0, s3", "\tbuffer_load_dwordx4 v2, s[0:3], 0 offen"]) == ([], 0)
    base = ["\tv_readfirstlane_b32 s5, v49", "\ts_mov_b32 m0, s9"]
    assert len(find_hazards([*base, "\ts_nop 2", "\tglobal_load_lds_dwordx4 v54, s[4:5] nt"])[0]) == 1
    assert find_hazards([*base, "\ts_nop 3", "\tglobal_load_lds_dwordx4 v54, s[4:5] nt"]) == ([], 1)
    assert find_hazards([*base, "\ts_nop 0", "\tglobal_load_dword v54, v1, s[6:7]"]) == ([], 0)
    assert len(find_hazards(["\tv_add_co_u32_e64 v0, s[2:3], v1, v2", "\tbuffer_load_dword v1, v0, s[8:11], s3 offen"])[0]) == 1


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
