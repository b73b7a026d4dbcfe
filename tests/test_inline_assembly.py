"""Inline assembly holds no memory instruction: the wait states between a
register's write and a memory instruction's read of it, and the waits for what
is in flight, are put in by the compiler for its own instructions only."""
import glob
import os
import re

from paper_2412_13547_amd import build

MEMORY = re.compile(r"\b(global|flat|buffer|scratch|s_load|s_buffer|tbuffer|ds)_\w+")


def test_no_memory_instruction_in_inline_assembly():
    files = glob.glob(os.path.join(build.CSRC, "*.hip")) + glob.glob(os.path.join(build.CSRC, "*.hpp"))
    assert len(files) > 5
    found = 0
    for path in files:
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
            found += 1
            block = text[m.end():text.index(";\n", m.end())]
            code = " ".join(re.findall(r'"((?:[^"\\]|\\.)*)"', block))
            assert not MEMORY.search(code), f"{os.path.basename(path)}: {code}"
    assert found > 0
