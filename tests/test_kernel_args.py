"""The kernel's argument segment can be addressed in the kernel itself only: in
a function that is called, not inlined, the compiler gives a null pointer
without a word.  Every function that reads the arguments there has to be
__forceinline__ (or the kernel)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_00976_amd", "csrc")


def test_kernel_args_only_where_inlined():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path, encoding="utf-8").read()
        heads = [(m.start(), m.group(0)) for m in re.finditer(r"^[^\n/]*\b(?:__device__|__global__)\b[^\n]*", text, re.M)]
        for use in re.finditer(r"\bkernel_args<", text):
            head = [h for at, h in heads if at < use.start()][-1]
            assert "__forceinline__" in head or "__global__" in head, (os.path.basename(path), head)
            seen += 1
    assert seen > 0
