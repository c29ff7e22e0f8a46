"""Alignment of the LDS arrays in the device sources: an array of floats or bytes that is
accessed 16 bytes at a time states that alignment (it is only its element's otherwise, and
where the compiler puts the array decides)."""
import os
import re

from conftest import ROOT

SRC = os.path.join(ROOT, "paper_1309_0052_amd", "csrc", "gnss_kernels.hip")
# arrays that carry 16-byte accesses through a pointer of another type
WIDE = {"s_stage": "k_corr_x", "smem": "k_corr"}


def test_arrays_with_wide_accesses_state_their_alignment():
    with open(SRC) as f:
        src = f.read()
    for name, kernel in WIDE.items():
        decl = re.findall(r"__shared__([^;\n]*?)\b(?:float|char)\s+%s\[" % name, src)
        assert decl, (kernel, name)
        assert all("__align__(16)" in d for d in decl), (kernel, name, decl)
