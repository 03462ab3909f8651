"""A check of the built library's own device code.

Where lanes rejoin after a divergent branch, a block restores exec first.  Under register pressure the
compiler has put a spill (a copy of a vector register to an accumulation register or to scratch) ahead of
that restore, next to its scalar spills: only the lanes that took the branch then store the value, and the
others read garbage later.  The results are wrong on some grids and months only, so the code is looked at."""

import os
import re
import shutil
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1410_0204_amd", "libtmm.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

INSTR = re.compile(r"^\t(.*?)\s*//\s*([0-9A-F]+):")
SPILL = re.compile(r"(v_accvgpr_write_b32 a\d+, v\d|v_accvgpr_mov|scratch_store|buffer_store_dword\S* .* s\[0:3\], 0 )")
LEAVES = re.compile(r"(s_cbranch|s_branch|s_endpgm|s_barrier|s_\w+_saveexec|s_\w+ exec)")


def spills_before_restore(lines):
    """(address, instruction) of every spill between a block that an execz branch leads to and the
    block's own restore of exec."""
    code = []
    targets = set()
    for line in lines:
        m = INSTR.match(line)
        if not m:
            continue
        addr, text = int(m.group(2), 16), m.group(1)
        code.append((addr, text))
        b = re.match(r"s_cbranch_execz (\d+)", text)
        if b:
            d = int(b.group(1))
            targets.add(addr + 4 + 4 * (d - 65536 if d >= 32768 else d))
    found = []
    for i, (addr, _) in enumerate(code):
        if addr not in targets:
            continue
        seen = []
        for k in range(i, len(code)):
            at, text = code[k]
            if text.startswith("s_or_b64 exec, exec"):
                found += seen
                break
            if LEAVES.match(text):
                break
            if SPILL.match(text):
                seen.append((at, text))
    return found


def test_the_check_finds_a_misplaced_spill():
    def asm(*instrs):
        return [f"\t{t} // {4096 + 4 * i:012X}: 00000000" for i, t in enumerate(instrs)]
    good = asm("s_and_saveexec_b64 s[2:3], vcc", "s_cbranch_execz 1", "v_mov_b32_e32 v1, v2",
               "v_writelane_b32 v254, s64, 61", "s_or_b64 exec, exec, s[2:3]", "v_accvgpr_write_b32 a26, v28")
    bad = asm("s_and_saveexec_b64 s[2:3], vcc", "s_cbranch_execz 1", "v_mov_b32_e32 v1, v2",
              "v_writelane_b32 v254, s64, 61", "v_accvgpr_write_b32 a26, v28", "s_or_b64 exec, exec, s[2:3]")
    assert spills_before_restore(good) == []
    assert [t for _, t in spills_before_restore(bad)] == ["v_accvgpr_write_b32 a26, v28"]


def test_no_spill_ahead_of_exec(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objs = sorted(tmp_path.glob("*gfx950"))
    assert len(objs) == 4
    for obj in objs:
        out = subprocess.run([OBJDUMP, "-d", str(obj)], check=True, capture_output=True, text=True).stdout
        lines = out.splitlines()
        assert len(lines) > 10000
        assert spills_before_restore(lines) == [], obj.name
