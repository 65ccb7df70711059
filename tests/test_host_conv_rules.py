"""The rules by which near_field = AUTO takes its transforms, on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_08509_amd", "csrc")


def _run(tmp_path, code):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include "conv_rules.hpp"\n#include <cstdio>\nusing namespace fep3m;\n' + code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()


def _coarsens(n):
    while n > 4 and n % 2 == 0:
        n //= 2
    while n > 6 and n % 3 == 0:
        n //= 3
    return n <= 16


def test_lattice_edges(tmp_path):
    """Every edge has two radices of the passes, a box's lattice keeps n_sr empty elements, periodic meshes that the
    multigrid hierarchy takes have a lattice up to 64 elements and none above."""
    out = _run(tmp_path, """int main() {
      for (int box = 0; box < 2; ++box) for (int s = 1; s <= 3; ++s) for (int n = 2 * s + 1; n <= 130; ++n) {
        int a = 0, b = 0; const int N = conv_edge(n, s, box);
        if (N) radices(N, a, b);
        std::printf("%d,%d,%d,%d,%d,%d ", box, s, n, N, a, b); } }""")
    radix = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 13}
    for box, s, n, N, a, b in (map(int, v.split(",")) for v in out):
        if n > 64:
            assert N == 0
        elif box:
            assert N >= n + s and N <= 72
        else:
            assert N in (0, n) and (N == n or not _coarsens(n))
        assert N == 0 or (a * b == N and {a, b} <= radix)


@pytest.mark.parametrize("spec,total,free,take", [
    (1, 2, 8, 1), (1, 2, 7.9, 0), (25, 26.6, 288, 1), (25, 26.6, 100, 0), (33, 34, 288, 0), (3, 80, 288, 0)])
def test_memory_rule(tmp_path, spec, total, free, take):
    """A quarter of the free memory at most, work arrays of a large batch included, and 32 GiB of spectrum."""
    g = lambda v: "size_t(%d)" % int(v * 2 ** 30)
    assert _run(tmp_path, 'int main() { std::printf("%%d", int(conv_memory(%s, %s, %s))); }' % (g(spec), g(total), g(free))) \
        == [str(take)]
