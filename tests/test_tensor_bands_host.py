"""The tensor set-up's distance bands do not depend on how the compiler
contracts sums of products (no GPU needed).

Two kernels write the offsets on either side of 40 h and each skips the
other's, so a disagreement would leave an offset unwritten.  The band function
they share is compiled for the host with contraction off and with contraction
on (fused multiply-add available) and must place every offset of cells with
many ties on the edges alike.  The plain sum of products, the planted mistake,
does not: the same two builds disagree on some offsets, so the test can fail.
"""

import os
import shutil
import subprocess

import pytest

from paper_1405_2728_amd import _build

SRC = r"""
#include <cstdio>
#define __host__
#define __device__
#include "mm_bands.h"
static int plain(double X, double Y, double Z, double h) {
  const double r2 = X * X + Y * Y + Z * Z;
  return r2 < 36.0 * h * h ? 0 : r2 < 256.0 * h * h ? 1 : r2 < 1600.0 * h * h ? 2 : 3;
}
int main() {
  const double cells[][3] = {{5e-9, 5e-9, 5e-9}, {3e-9, 3e-9, 3e-9}, {4e-9, 5e-9, 3e-9},
                             {7e-9, 7e-9, 3.5e-9}, {1e-8 / 3, 1e-8 / 3, 1e-8 / 3}};
  for (auto& d : cells) {
    const double h = d[0] > d[1] ? (d[0] > d[2] ? d[0] : d[2]) : (d[1] > d[2] ? d[1] : d[2]);
    for (int i = 0; i < 48; ++i)
      for (int j = 0; j < 48; ++j)
        for (int k = 0; k < 48; ++k) {
          const double X = i * d[0], Y = j * d[1], Z = k * d[2];
          std::putchar('0' + mmk::offset_band(X, Y, Z, h));
          std::putchar('0' + plain(X, Y, Z, h));
        }
  }
}
"""


def test_bands_do_not_depend_on_contraction(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None or os.uname().machine != "x86_64":
        pytest.skip("no x86-64 C++ compiler")
    if " fma " not in open("/proc/cpuinfo").read():
        pytest.skip("no fused multiply-add on this machine")
    src = tmp_path / "bands.cpp"
    src.write_text(SRC)
    out = {}
    for mode in ("off", "fast"):
        exe = tmp_path / mode
        subprocess.run([cxx, "-O2", "-std=c++17", "-mfma", "-ffp-contract=" + mode,
                        "-I" + os.path.join(_build.HERE, "csrc"), "-o", str(exe), str(src)],
                       check=True)
        out[mode] = subprocess.run([str(exe)], capture_output=True, check=True).stdout
    assert len(out["off"]) == 2 * 5 * 48 ** 3
    assert out["off"][0::2] == out["fast"][0::2]          # offset_band
    assert out["off"][1::2] != out["fast"][1::2]          # the plain sum
    assert set(out["off"][0::2]) == set(b"0123")


def test_the_kernels_take_their_bands_from_it():
    text = open(os.path.join(_build.HERE, "csrc", "tensor.hip")).read()
    split = text[text.index("k_newell_near("):text.index("k_embed_thin(")]
    assert split.count("offset_band(") == 2
    assert "1600.0" not in split and "256.0" not in split and "36.0" not in split
