"""Registers and shared memory of the compiled pair kernels (csrc/kernels_pair.hpp),
read from the kernel descriptors of the built library, and the rules that cut a
field into slabs, evaluated on the host.

An instance that keeps values in scratch memory pays for them at every item.
The split by cutoff shell (BINS) once held its eight FP64 bins in registers
through all transforms of an item and spilled up to 184 bytes per lane; its
instances are held to what a handful of spilled registers takes.  On the 36
grid it once missed a second workgroup per CU by 32 bytes of shared memory,
counted with a constant that was too small.
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


HOST = r"""
#include <cstdio>
#include "kernels_pair.hpp"
using namespace ltmp2;
template <int... N> void all(std::integer_sequence<int, N...>) {
  auto grid = [](int n) {
    for (int es : {4, 8})
      for (int k = 1; k <= pair_kf(n); ++k) {
        if (k < pair_kw(n) - 1 || (k > pair_kw(n) && k < pair_kf(n))) continue;
        for (int bins : {0, 1})
          for (int ns = 1; ns <= n; ++ns)
            if (n % ns == 0)
              printf("%d %d %d %d %d %d %d %zu %zu\n", es, n, k, bins, ns,
                     ns == pair_slabs(es, n, k, bins), pair_threads(es, n, k),
                     pair_lds_bytes(es, n, k, ns, pair_cols_max(k)),
                     pair_static(k, pair_threads(es, n, k), bins));
      }
  };
  (grid(N), ...);
}
int main() { all(std::integer_sequence<int, GRIDS_>{}); }
"""


@pytest.fixture(scope="module")
def slabs(tmp_path_factory):
    """{(element size, n, k, bins): [(slabs, chosen, threads, dynamic, static bytes)]}"""
    from paper_1611_06797_amd.build import CSRC, GRIDS, HIPCC
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("slabs")
    (d / "t.hip").write_text(HOST.replace("GRIDS_", ", ".join(map(str, GRIDS))))
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++20", "-w", f"-I{CSRC}", "-o", d / "t",
                    d / "t.hip"], check=True, capture_output=True)
    out = {}
    for line in subprocess.run([d / "t"], check=True, capture_output=True,
                               text=True).stdout.splitlines():
        v = [int(x) for x in line.split()]
        out.setdefault(tuple(v[:4]), []).append(tuple(v[4:]))
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (scratch bytes per lane, static shared memory)}"""
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
            out[name] = tuple(int(re.search(rf"\.{q}_segment_fixed_size:\s+(\d+)", entry).group(1))
                              for q in ("private", "group"))
    return out


@pytest.mark.parametrize("bins", [0, 1])
def test_pair_instances_spill_a_few_registers_at_most(kernels, bins):
    pair = {n: s[0] for n, s in kernels.items()
            if re.search(rf"k_pairI[df]Li\d+ELi\d+ELb{bins}E", n)}
    assert len(pair) >= 2 * 12 * 2  # two types, twelve grids, two or three kept sets
    # twelve 32-bit registers of the 64 to 256 an instance has
    assert {n: s for n, s in pair.items() if s > 48} == {}


def test_static_shared_memory_is_counted(kernels, slabs):
    seen = 0
    for name, (_, static) in kernels.items():
        m = re.search(r"k_pairI([df])Li(\d+)ELi(\d+)ELb([01])E", name)
        if not m:
            continue
        key = (8 if m[1] == "d" else 4, int(m[2]), int(m[3]), int(m[4]))
        ns, _, nt, lds, counted = [x for x in slabs[key] if x[1]][0]
        # at most the row table, which one slab does without, and 64 bytes of alignment too many
        assert static <= counted <= static + 4 * (2 * key[2] + 1) + 64, key
        half = [x for x in slabs[key] if x[3] + static <= 80 * 1024]
        if key[0] == 4 and half:  # FP32: never one workgroup per CU where two would fit
            assert lds + static <= 80 * 1024, key
        assert lds <= 150 * 1024 and nt % 64 == 0 and nt <= 512, key
        seen += 1
    assert seen >= 48


def test_slabs_keep_their_threads_busy(slabs):
    """A field is not cut so thin that a slab's z lines leave most of its threads idle: FP64
    fields of the 25, 27 and 30 grids once went in five to fifteen slabs of 60 to 125 lines."""
    for key, rows in slabs.items():
        ns, _, nt, lds, _ = [x for x in rows if x[1]][0]
        lines = key[1] // ns * key[1]
        fewer = [x for x in rows if x[0] < ns and x[3] <= 150 * 1024]
        if fewer:  # more slabs than shared memory asks for
            assert lines * 100 >= 60 * -(-lines // nt) * nt, (key, ns, nt)
