"""CPU test of the inline assembly in the HIP sources: a statement that writes m0 says so, as the compiler
may keep a value of its own there (for its own loads to shared memory, register indexing, messages)."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WRITES_M0 = re.compile(r"\bs_\w+\s+m0\s*,")


def test_m0_is_declared():
    found = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2608_22704_amd", "csrc", "*.h*"))):
        src = open(path).read()
        for m in re.finditer(r"__asm__\s+(?:volatile\s*)?\((.*?)\);", src, re.S):
            if WRITES_M0.search(m.group(1)):
                found += 1
                assert '"m0"' in m.group(1).rsplit(":", 1)[1], f"{os.path.basename(path)}: {m.group(0)}"
    assert found
