"""The reciprocal square root of the boxes' near sums: full float64 length
from any estimate as good as the hardware's, and the values of 1 / sqrt at
zero and infinity.  The refinement is host code too, compiled here."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_08509_amd", "csrc")

CODE = r"""
#include "rsqrt_step.hpp"
#include <cmath>
#include <cstdio>
#include <random>
int main() {
  std::mt19937_64 g(3);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long double worst = 0.0L;
  for (int i = 0; i < 2000000; ++i) {
    const double x = i & 1 ? 1.0 + 3.0 * u(g) : std::exp(-20.0 + 24.0 * u(g));
    const long double r = 1.0L / sqrtl((long double)x);
    const double d = (i % 7 ? 2.0 * u(g) - 1.0 : (i & 2 ? 1.0 : -1.0)) * 1.2e-7;   // estimate good to 2^-23
    const long double e = fabsl(((long double)fep3m::rsqrt_step3(x, double(r * (1.0L + d))) - r) / r);
    if (e > worst) worst = e;
  }
  const double inf = INFINITY;
  std::printf("%.6Le %d %d %d", worst, fep3m::rsqrt_step3(0.0, inf) == inf, fep3m::rsqrt_step3(inf, 0.0) == 0.0,
              std::isnan(fep3m::rsqrt_step3(NAN, NAN)));
}
"""


def test_refined_reciprocal_root_has_full_length(tmp_path):
    """Half a unit in the last place of the result (2^-53) and half of the rounding of x y (2^-54) bound the error:
    1.7e-16.  1 / sqrt(x) by a square root and a division is within 2^-52."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(CODE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    worst, zero, inf, nan = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert float(worst) <= 2.0 ** -53 + 2.0 ** -54 + 1e-19
    assert (zero, inf, nan) == ("1", "1", "1")


def test_boxes_take_full_length_roots():
    src = open(os.path.join(CSRC, "k_box.hip")).read()
    assert "rsqrt_pos(" not in src and "builtin_amdgcn_rsq" not in src
