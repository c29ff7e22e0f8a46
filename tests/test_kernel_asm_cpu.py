"""Inline assembly in the device sources: only empty statements and counter waits.

The compiler inserts the wait states that gfx950 needs between dependent vector
instructions (three between a dot product and another kind of instruction that
reads its result) for instructions that it generates.  It does not look into an asm
string, so an arithmetic instruction written there is without them, wherever the
scheduler happens to put its reader.
"""
import glob
import os
import re

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1309_0052_amd", "csrc")


def test_inline_assembly_holds_no_arithmetic():
    found = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            src = f.read()
        for m in re.finditer(r'\basm\b(?:\s+volatile)?\s*\(\s*"([^"]*)"', src):
            for ins in re.split(r"\\n|;", m.group(1)):
                if ins.strip() and not ins.strip().startswith("s_waitcnt"):
                    found.append("%s:%d: %s" % (os.path.basename(path), src.count("\n", 0, m.start()) + 1, ins.strip()))
    assert not found, found
