"""Wait state between a write of M0 and the LDS copy that reads it, in the built gfx950 code.

gfx9 needs one instruction (an s_nop or any other) between a scalar write of M0 and a
global_load_lds, which takes its LDS address from M0.  The compiler inserts it for its own copies but
cannot see into inline asm, where all of this library's copies are issued.
"""
import os
import re
import shutil
import subprocess

from paper_2609_38795_amd import binding, build

BIN = "/opt/rocm/llvm/bin"


def _disassembly(tmp_path):
    binding.load_library()
    lib = shutil.copy(build.LIB, tmp_path)
    objdump = os.path.join(BIN, "llvm-objdump")
    subprocess.run([objdump, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    code = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(code) == 1, code
    res = subprocess.run([objdump, "-d", "--no-show-raw-insn", os.path.join(tmp_path, code[0])],
                         check=True, capture_output=True, text=True)
    return [line.split("//")[0].strip() for line in res.stdout.splitlines()]


def unguarded_copies(lines):
    """(copies, those whose preceding instruction writes M0) of a listing."""
    copies, bad, last = 0, [], ""
    for line in lines:
        if not line or line.endswith(":"):
            continue
        if re.match(r"(global|buffer|scratch)_load_lds|buffer_load.*\blds\b", line):
            copies += 1
            if re.match(r"s_\w+ m0\b", last):
                bad.append((last, line))
        last = line
    return copies, bad


def test_rule_finds_an_unguarded_copy():
    good = ["s_mov_b32 m0, s1", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]"]
    assert unguarded_copies(good) == (1, [])
    assert len(unguarded_copies([good[0], good[2]])[1]) == 1


def test_no_copy_follows_the_write_of_its_m0(tmp_path):
    copies, bad = unguarded_copies(_disassembly(tmp_path))
    assert copies > 0
    assert not bad, f"{len(bad)} of {copies} copies, first: {bad[0]}"
