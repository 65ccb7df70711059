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


# (one-element or 27-element, q, elements, n_sr, configurations, box): near field and moment adjoint of the
# transforms and of the table sums, ms
TIMES = [
    ("one", 3, 16, 1, 16, 1, 1.061, 0.516), ("one", 3, 16, 1, 1, 1, 0.164, 0.342), ("one", 4, 16, 1, 16, 0, 2.719, 1.866),
    ("one", 4, 16, 1, 1, 0, 0.287, 1.073), ("27", 1, 16, 1, 16, 0, 0.287, 0.161), ("27", 1, 16, 1, 1, 0, 0.088, 0.109),
    ("27", 4, 16, 1, 16, 0, 14.27, 7.01), ("27", 4, 16, 1, 1, 0, 1.142, 3.856), ("27", 1, 64, 1, 1, 0, 0.763, 0.519),
    ("27", 4, 40, 1, 1, 0, 12.58, 6.49), ("one", 3, 40, 1, 1, 0, 0.669, 0.516), ("one", 3, 27, 1, 1, 0, 0.300, 0.411),
    ("one", 2, 8, 1, 128, 1, 0.640, 0.583), ("27", 2, 8, 1, 128, 0, 0.998, 0.701), ("27", 3, 5, 1, 1000, 0, 5.303, 13.64),
    ("one", 3, 3, 1, 1000, 1, 1.266, 0.855), ("one", 3, 8, 2, 256, 1, 3.750, 2.919), ("one", 3, 8, 2, 16, 1, 0.286, 0.977),
    ("one", 3, 16, 2, 32, 1, 2.349, 2.974), ("27", 1, 8, 2, 256, 0, 0.742, 0.862), ("one", 3, 8, 3, 256, 1, 5.380, 7.103),
    ("27", 4, 64, 3, 1, 0, 48.1, 321.0), ("27", 1, 8, 3, 256, 0, 0.744, 2.179)]


def test_faster_path(tmp_path):
    """The rule takes the faster of the two paths at measured points on both sides of each of its lines."""
    args = []
    for sup, q, n, nsr, nb, box, _, _ in TIMES:
        args.append("{%d,%d,%d,%d,%d,%d}" % (n, nsr, q + 2, q + 1 if sup == "27" else q - 1, box, nb))
    out = _run(tmp_path, "int main() { int c[][6] = {" + ",".join(args) + "};\n"
               "for (auto &v : c) std::printf(\"%d \", int(conv_pays(v[0], conv_edge(v[0], v[1], v[4]), v[1], v[2], v[3], v[4], v[5]))); }")
    for t, took in zip(TIMES, out):
        assert int(took) == (t[6] < t[7]), t
