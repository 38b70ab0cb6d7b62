"""The stored HBM traffic of the pair kernel is reported only while its sources are
unchanged: the hash covers every file the kernel is compiled from and the files
that launch it and choose its work list and block size.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1611_06797_amd", "csrc")


def _included(name, seen):
    if name in seen or not os.path.exists(os.path.join(CSRC, name)):
        return seen
    seen.add(name)
    with open(os.path.join(CSRC, name)) as f:
        for inc in re.findall(r'#include "([^"]+)"', f.read()):
            _included(inc, seen)
    return seen


def test_pair_sources_cover_the_kernel():
    import bench
    need = _included("kernels_pair.hpp", set()) | {"grid_kernels.hip", "ltmp2.hip"}
    assert {"fft.hpp", "rfft.hpp", "transforms.hpp"} <= need
    assert need <= set(bench.PAIR_SOURCES)
    for f in bench.PAIR_SOURCES:
        assert os.path.exists(os.path.join(CSRC, f)), f
