"""Host check of the register FFTs of real lines (csrc/rfft.hpp), as tests/test_fft_host.py
checks the complex ones: every length that a compiled grid or a factor of one
uses, against numpy's real FFT, FP64 and FP32, with the same bounds (the real
transform does a part of the complex one's operations).
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

from tests.test_fft_host import ROOT, SIZES

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "rfft.hpp"
using namespace ltmp2;
template <class T, int N> void one(FILE* in, FILE* out) {
  T x[N];
  cplx<T> X[N / 2 + 1];
  for (int k = 0; k < N; ++k) { double a; if (fscanf(in, "%lf", &a) != 1) exit(2); x[k] = T(a); }
  RFft<T, N>::run(x, X);
  for (int k = 0; k <= N / 2; ++k) fprintf(out, "%.17g %.17g\n", double(X[k].x), double(X[k].y));
}
template <class T> void all(FILE* in, FILE* out) {
#define S_(n) one<T, n>(in, out);
  SIZES_
}
int main(int argc, char** argv) {
  FILE* in = fopen(argv[1], "r"); FILE* out = fopen(argv[2], "w");
  all<double>(in, out); all<float>(in, out);
  fclose(in); fclose(out); return 0;
}
"""


def test_real_register_ffts_match_numpy(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(
        "#pragma once\n#define __host__\n#define __device__\n#define __forceinline__ inline\n")
    sizes = [1] + SIZES
    (tmp_path / "t.cpp").write_text(SRC.replace("SIZES_", " ".join(f"S_({n})" for n in sizes)))
    subprocess.run([gxx, "-std=c++20", "-O1", f"-I{tmp_path}",
                    f"-I{os.path.join(ROOT, 'paper_1611_06797_amd', 'csrc')}", "-o",
                    str(tmp_path / "t"), str(tmp_path / "t.cpp")], check=True, capture_output=True)
    rng = np.random.default_rng(12)
    lines = [rng.uniform(-1, 1, n) for n in sizes]
    text = "".join(f"{float(x)!r}\n" for ln in lines for x in ln)
    (tmp_path / "in.txt").write_text(text + text)
    subprocess.run([str(tmp_path / "t"), str(tmp_path / "in.txt"), str(tmp_path / "out.txt")],
                   check=True)
    vals = np.loadtxt(tmp_path / "out.txt")
    out = vals[:, 0] + 1j * vals[:, 1]
    pos = 0
    for prec, tol in (("f64", 1e-13), ("f32", 3e-6)):
        for x in lines:
            ref = np.fft.rfft(x)
            got = out[pos:pos + len(ref)]
            pos += len(ref)
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (prec, len(x))
    assert pos == len(out)
