"""The tables behind the transforms' spectrum are symmetric under the axis
reflections to the last bit (the spectrum is stored for one octant).  The
host sources are compiled into a small program here."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_08509_amd", "csrc")

CODE = r"""
#include "host_tables.hpp"
#include "table_symmetry.hpp"
#include <cmath>
#include <cstdio>
#include <cstdlib>
using namespace fep3m;
int main(int, char **v) {
  const int q = std::atoi(v[1]), support = std::atoi(v[2]), nsr = std::atoi(v[3]), p = q + 2, q1 = p + 1, S = 2 * nsr + 1;
  const Screen1D scr = make_screen(q, support);
  const int nl = scr.d + 1;
  Vec T;
  compute_tables(p, scr, nsr, 2 * nsr + 3, T);
  Vec U = T;
  for (std::size_t k = U.size(); k-- > 0;) symmetrise_entry(k, p, nl, nsr, U.data());
  double big = 0.0, moved = 0.0, before = 0.0;
  long wrong = 0;
  std::size_t i = 0;
  for (int az = 0; az < nl; ++az) for (int ay = 0; ay < nl; ++ay) for (int ax = 0; ax < nl; ++ax)
  for (int dz = 0; dz < S; ++dz) for (int dy = 0; dy < S; ++dy) for (int dx = 0; dx < S; ++dx)
  for (int mz = 0; mz < q1; ++mz) for (int my = 0; my < q1; ++my) for (int mx = 0; mx < q1; ++mx, ++i) {
    big = std::fmax(big, std::fabs(T[i]));
    moved = std::fmax(moved, std::fabs(U[i] - T[i]));
    for (int r = 1; r < 8; ++r) {
      auto at = [&](int d, int n, int b) { return (r >> b & 1) ? n - 1 - d : d; };
      const std::size_t a = ax + nl * (ay + std::size_t(nl) * az);
      const std::size_t D = at(dx, S, 0) + S * (at(dy, S, 1) + std::size_t(S) * at(dz, S, 2));
      const std::size_t m = at(mx, q1, 0) + q1 * (at(my, q1, 1) + std::size_t(q1) * at(mz, q1, 2));
      const double sg = ((r & ax) ^ (r >> 1 & ay) ^ (r >> 2 & az)) & 1 ? -1.0 : 1.0;
      const std::size_t j = (a * S * S * S + D) * q1 * q1 * q1 + m;
      if (sg * U[j] != U[i]) ++wrong;
      before = std::fmax(before, std::fabs(sg * T[j] - T[i]));
    }
  }
  std::printf("%ld %.3e %.3e %zu %zu", wrong, moved / big, before / big, i, T.size());
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("sym")
    (d / "t.cpp").write_text(CODE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I" + CSRC, str(d / "t.cpp"),
                    os.path.join(CSRC, "host_tables.cpp"), os.path.join(CSRC, "host_fe.cpp"), "-o", str(d / "t")],
                   check=True)
    return str(d / "t")


@pytest.mark.parametrize("q,support,nsr", [(2, 0, 1), (3, 0, 1), (4, 0, 1), (1, 1, 2), (2, 1, 1), (3, 1, 1)])
def test_symmetrised_tables_are_symmetric(program, q, support, nsr):
    wrong, moved, before, n, size = subprocess.run([program, str(q), str(support), str(nsr)], capture_output=True,
                                                   text=True, check=True).stdout.split()
    assert int(wrong) == 0 and n == size
    # an average of eight values of which no two differ by more than `before`
    assert float(moved) <= float(before) < 1e-13
