"""Registers of the compiled pair kernels (csrc/kernels_pair.hpp), read from the
kernel descriptors of the built library.

An instance that keeps values in scratch memory pays for them at every item.
The split by cutoff shell (BINS) once held its eight FP64 bins in registers
through all transforms of an item and spilled up to 184 bytes per lane; its
instances are held to what a handful of spilled registers takes.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1611_06797_amd", "libltmp2.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: scratch bytes per lane}"""
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("no LLVM tools")
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("objects")
    lib = shutil.copy(LIB, d / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True,
                   capture_output=True, cwd=d)
    out = {}
    for f in glob.glob(str(d / "*gfx950*")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f], check=True,
                               capture_output=True, text=True).stdout
        for entry in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            out[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry).group(1))
    return out


@pytest.mark.parametrize("bins", [0, 1])
def test_pair_instances_spill_a_few_registers_at_most(kernels, bins):
    pair = {n: s for n, s in kernels.items()
            if re.search(rf"k_pairI[df]Li\d+ELi\d+ELb{bins}E", n)}
    assert len(pair) >= 2 * 12 * 2  # two types, twelve grids, two or three kept sets
    # twelve 32-bit registers of the 64 to 256 an instance has
    assert {n: s for n, s in pair.items() if s > 48} == {}
