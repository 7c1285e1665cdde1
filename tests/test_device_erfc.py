"""The erfc of the flux kernels (common.h: a polynomial of erf for |x| <= 1,
beyond it exp(-x^2) times a polynomial of the scaled complement) on the
host, where the same functions compile, against the C library's erfc.

Bars, in units of the type's 2^-52 or 2^-23: 4 absolute everywhere (the
value is at most 2, and |x| <= 1 and the negative side subtract from 1 or
2); on the positive tail (2 x^2 + 16) relative: exp(-x^2) carries the
rounding of x^2 (x^2 units) on both sides of the comparison, the polynomial,
the reciprocal and the products the rest."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r'''
#include "paper_1909_01580_amd/csrc/common.h"
#include <cmath>
#include <cstdio>
template <typename T>
static bool check(double unit, double top) {
  bool ok = true;
  for (int i = -200000; i <= 200000; ++i) {
    const T x = T(top * i / 200000.0);
    const T e = std::exp(-x * x);
    const double v = (double)hgks::d_erfc<T>(x, e), r = std::erfc((double)x);
    if (!(std::fabs(v - r) <= 4 * unit)) ok = false;
    if (x > 1 && r > 1e-30 && !(std::fabs(v - r) <= (2.0 * x * x + 16) * unit * r)) ok = false;
    if (!ok) { printf("x %.17g value %.17g erfc %.17g\n", (double)x, v, r); return false; }
  }
  // the branches meet, and far arguments give exactly 0 and 2
  for (T x : {T(1), std::nextafter(T(1), T(2)), T(-1), std::nextafter(T(-1), T(-2))})
    if (std::fabs((double)hgks::d_erfc<T>(x, std::exp(-x * x)) - std::erfc((double)x)) > 4 * unit) return false;
  if (hgks::d_erfc<T>(T(1e6), T(0)) != T(0) || hgks::d_erfc<T>(T(-1e6), T(0)) != T(2)) return false;
  const T nan = std::nan("");
  return std::isnan((double)hgks::d_erfc<T>(nan, nan));
}
int main() {
  if (!check<double>(0x1p-52, 12.0) || !check<float>(0x1p-23, 8.0)) return 1;
  printf("ok\n");
  return 0;
}
'''


def test_erfc_against_the_c_library(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src = tmp_path / "erfc.hip"
    src.write_text(HARNESS)
    exe = str(tmp_path / "erfc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", ROOT, "-o", exe, str(src)],
                   check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
