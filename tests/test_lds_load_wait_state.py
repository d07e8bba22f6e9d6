"""CPU-only: a load to LDS takes its destination from M0, and gfx9 asks for one wait state between a scalar write of M0 and such a load.  The
compiler inserts it into its own code but not into inline assembly, so every instruction sequence written by hand has to hold one."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_08245_amd", "csrc")


def _sequences():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"(?:__asm__|asm)\s+(?:volatile\s*)?\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m[1]))
            yield os.path.basename(path), [i.strip() for i in re.split(r"\\n\\t|\\n", body) if i.strip()]


def test_one_instruction_between_m0_and_a_load_to_lds():
    found = 0
    for name, instructions in _sequences():
        for before, after in zip(instructions, instructions[1:]):
            if re.match(r"s_\w+\s+m0\s*,", before):
                found += 1
                assert not re.search(r"\blds\b|_lds_", after), f"{name}: {before}; {after}"
        for i in instructions:                     # the write of M0 belongs into the same sequence as the load
            if re.search(r"\blds\b|load_lds_", i):
                assert any(re.match(r"s_\w+\s+m0\s*,", j) for j in instructions), f"{name}: {i}"
    assert found >= 6
