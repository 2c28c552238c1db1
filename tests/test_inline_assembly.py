"""Rules for inline assembly that the compiler cannot check (it does not look into a statement's text).

A statement that writes m0 has to name it, or the compiler may keep a value of its own there.  And the hardware does not wait for
a scalar register that a vector instruction has just written (v_readlane restores spilled ones) when a memory
instruction takes its address from it: five wait states have to lie between, which the compiler inserts for its own
instructions only.
"""
import glob
import os
import re

from paper_2510_26475_amd import build

SOURCES = sorted(glob.glob(os.path.join(build.CSRC, "*.h*")))


def _statements():
    for path in SOURCES:
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"asm volatile\((.*?)\);", text, flags=re.S):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1).split(":")[0])).replace("\\n", "\n").replace("\\t", " ")
            yield os.path.basename(path), code, m.group(1)


def test_there_are_statements_to_look_at():
    assert sum("global_load_lds" in code for _, code, _ in _statements()) == 1


def test_statements_that_write_m0_name_it():
    for path, code, whole in _statements():
        if re.search(r"\bs_\w+ m0\b", code):
            assert '"m0"' in whole.split(":")[-1], (path, code)


def test_memory_instructions_wait_for_their_scalar_address():
    for path, code, whole in _statements():
        lines = [line.strip() for line in code.splitlines()]
        for i, line in enumerate(lines):
            if re.match(r"(global|buffer|scratch)_", line) and re.search(r'"=?&?s"\(', whole):
                base = re.findall(r"%\d+", line)[-1]
                moved = any(re.match(rf"s_mov_b64 {base},", x) for x in lines[:i])   # (written by a scalar instruction)
                states = sum(int(x.split()[1]) + 1 if x.startswith("s_nop") else 1 for x in lines[:i])
                assert moved or states >= 5, (path, code)
                if "_lds_" in line:                                                  # m0: one wait state
                    assert not lines[i - 1].startswith("s_mov_b32 m0"), (path, code)
