"""A kernel's name says which kernel it is: no two of the library share one (a
profile lists them by name alone)."""
import collections
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2107_11810_amd", "csrc")
KERNEL = re.compile(r"__global__\s+void\s+(?:__launch_bounds__\((?:[^()]|\((?:[^()]|\([^()]*\))*\))*\)\s*)?(\w+)\s*\(")


def test_kernel_names_are_unique():
    names = collections.Counter()
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        found = KERNEL.findall(text)
        assert len(found) == text.count("__global__ "), path
        names.update(found)
    assert len(names) > 40
    assert [n for n, k in names.items() if k > 1] == []
