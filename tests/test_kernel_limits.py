"""Limits that the library sets for a kernel belong to the process."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_03641_amd", "csrc")


def test_lds_limits_are_constants():
    """A kernel's limit of dynamic LDS holds for every handle of the process, so
    none sets it from its own sizes: a constant expression, no call or member of
    an object.  (A runtime that enforces the limit would refuse the launches of
    the handles with larger blocks; not every one does.)"""
    found = 0
    for f in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(f) as src:
            text = src.read()
        for m in re.finditer(r"hipFuncAttributeMaxDynamicSharedMemorySize,([^;]*);", text):
            value = re.sub(r"\((int|size_t)\)", "", m.group(1)).rstrip().rstrip(")")
            found += 1
            assert re.fullmatch(r"[\s\w:*+]+", value), (os.path.basename(f), value)
    assert found >= 2
