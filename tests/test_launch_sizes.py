"""Launches of the work-list kernels stay below HIP's limit of 2^32 threads.

One workgroup per item is as many threads as items times workgroup size: cells
with many occupied states reach 2^32 within one block of outer vectors.  The
host library runs here against a stand-in for the HIP runtime that only notes
its launches; the ranges themselves are walked with the functions that the
kernels and the launchers share.
"""
import os
import shutil
import subprocess

import pytest

from tests import fake_hip

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# a cell of n_occ occupied and n_vir virtual orbitals, one plane wave each
CELL = """
def cell(L_, n, ecut, no, nst):
    import math
    b = 2 * math.pi / L_
    k = int(math.sqrt(2 * ecut) / b) + 1
    r = np.arange(-k, k + 1)
    m = np.stack([a.ravel() for a in np.meshgrid(r, r, r, indexing="ij")], axis=1)
    m = m[0.5 * b * b * (m * m).sum(1) < ecut].astype(np.int32)
    pos = m[(m[:, 0] > 0) | ((m[:, 0] == 0) & ((m[:, 1] > 0) | ((m[:, 1] == 0) & (m[:, 2] > 0))))]
    at = {tuple(v): i for i, v in enumerate(m.tolist())}
    c = np.zeros((nst, len(m)), complex)
    for s in range(nst):
        v = tuple(pos[s // 2].tolist())
        c[s, at[v]] = np.sqrt(0.5) * (1j if s % 2 else 1)
        c[s, at[tuple(-x for x in v)]] = np.conj(c[s, at[v]])
    e = np.concatenate([np.linspace(-1, -0.5, no), np.linspace(0.5, 2, nst - no)])
    return dict(L=L_, n_fft=n, ecut=ecut, eaux=5.0, miller=m, eps=e, coeff=c, n_occ=no, n_tau=1,
                tau=np.array([1.0]), w=np.array([1.0]))
"""
CONTEXT = """
d = cell({L}, {n}, {ecut}, {no}, {nst})
c = L.Context(d["L"], d["n_fft"], d["ecut"], {eaux}, d["miller"], d["eps"], d["coeff"],
              d["n_occ"], 1, tau=d["tau"], w=d["w"], prec={prec})
c.exchange(0, 0, {count} or c.info.g_block)
i = c.info
print(json.dumps(dict(n_grid=i.n_grid, pairs=i.n_occ * (i.n_occ + 1) // 2, block=i.g_block,
                      products=i.n_occ * i.n_vir)))
"""
BATCH = """
d = cell({L}, {n}, 7.2, {no}, {nst})
b = L.Batch([d], prec=L.BF16X3)
b.energy()
i = b.cell_info(0)
print(json.dumps(dict(n_grid=i.n_grid, pairs=i.n_occ * (i.n_occ + 1) // 2, block=i.n_h)))
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    d = tmp_path_factory.mktemp("fakehip")
    return fake_hip.build(d), d


def _check(lines, kernel):
    launches = [l for l in lines if l[0] == "launch"]
    assert launches
    for l in launches:
        assert int(l[2]) * int(l[5]) < 1 << 32, l
    mine = [l for l in launches if kernel in l[1]]
    return sum(int(l[2]) for l in mine), int(mine[0][5]), len(mine)


@pytest.mark.parametrize("no,prec", [(520, 1), (520, 2), (40, 1)])
def test_one_block_of_a_context(fake, no, prec):
    lines, (info,) = fake_hip.run(*fake, CELL + CONTEXT.format(
        L=18.0, n=30, ecut=7.2, eaux=5.0, no=no, nst=no + 30, prec=prec, count=0))
    assert info["n_grid"] == 30
    items = info["pairs"] * info["block"]
    blocks, nt, count = _check(lines, "6k_pairI")
    assert items <= blocks < items + 8 * count and count == 1 + (items * nt >= 1 << 32)


@pytest.mark.parametrize("L,n,no", [(18.0, 30, 260), (16.0, 27, 420)])
def test_one_round_of_a_batch(fake, L, n, no):
    lines, (info,) = fake_hip.run(*fake, CELL + BATCH.format(L=L, n=n, no=no, nst=no + 30))
    assert info["n_grid"] == n
    items = info["pairs"] * info["block"]
    blocks, _, count = _check(lines, "k_pair_multi")
    assert items <= blocks < items + 8 * count


def test_overlap_densities(fake):
    lines, (info,) = fake_hip.run(*fake, CELL + CONTEXT.format(
        L=20.0, n=36, ecut=7.5, eaux=0.8, no=2400, nst=5900, prec=1, count=1), timeout=300)
    blocks, nt, count = _check(lines, "k_real_forward")
    assert info["products"] <= blocks and info["products"] * nt >= 1 << 32 and count >= 2


HOST = r"""
#include <cstdio>
#include <vector>
#include "launch_items.hpp"
using namespace ltmp2;
int main() {
  for (int nt = 64; nt <= 512; nt += 64) {
    const long m = launch_items(nt);
    if (m % 8 || m * nt >= 1L << 32 || (m + 8) * nt < 1L << 32) return 1;
    for (long total : {0L, 1L, 7L, 8L, m - 1, m, m + 1, 2 * m, 3 * m + 5}) {
      long next = 0, n = 0;
      const int s = launch_ranges(total, nt, [&](long first, long count) {
        if (first != next || long(launch_blocks(count)) * nt >= 1L << 32) return 2;
        if (launch_blocks(count) < count || launch_blocks(count) % 8) return 3;
        next = first + count;
        ++n;
        return 0;
      });
      if (s || next != total || n != (total <= m ? 1 : (total + m - 1) / m)) return 4;
    }
  }
  for (long count : {1L, 7L, 8L, 9L, 63L, 64L, 1000L, 4097L}) {  // every item once
    std::vector<int> seen(count, 0);
    for (unsigned b = 0; b < launch_blocks(count); ++b) {
      const long t = block_item(b, count);
      if (t >= count) return 5;
      if (t >= 0) ++seen[t];
    }
    for (int x : seen)
      if (x != 1) return 6;
  }
  if (launch_ranges(100L, 64, [](long, long) { return 9; }) != 9) return 7;
  return 0;
}
"""


def test_ranges_cover_every_item_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "t.cpp").write_text(HOST)
    subprocess.run([gxx, "-std=c++20", "-O1", "-Wall", "-Werror",
                    f"-I{os.path.join(ROOT, 'paper_1611_06797_amd', 'csrc')}", "-o",
                    str(tmp_path / "t"), str(tmp_path / "t.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "t")]).returncode == 0
