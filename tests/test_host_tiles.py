"""Index rules of the tiled mesh kernels, on the CPU: the headers that hold
them are host code too and are compiled into a small program here."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1503_08509_amd", "csrc")


def _run(tmp_path, code):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()


def _levels(n):
    """Pairs (fine, coarse) of the order-1 levels below a mesh of n elements per axis."""
    out = []
    while n > 4 and n % 2 == 0:
        out.append((n, n // 2))
        n //= 2
    while n > 6 and n % 3 == 0:
        out.append((n, n // 3))
        n //= 3
    return out


@pytest.mark.parametrize("kind", ["restrict", "prolong"])
def test_transfer_tiles_stay_on_the_mesh(tmp_path, kind):
    """Every column that a tile of the order-1 transfers reads is an index of the axis, and the true periodic
    one wherever a coarse (restriction) or fine (prolongation) node of the mesh depends on it: on each pair of
    levels that a hierarchy of 3 to 512 elements holds, also where the tile is wider than the mesh."""
    pairs = sorted({p for n in range(3, 513) for p in _levels(n)})
    tile = {("restrict", 2): 7, ("restrict", 3): 4, ("prolong", 2): 8, ("prolong", 3): 5}
    calls = []
    for nf, nc in pairs:
        r = nf // nc
        te = tile[kind, r]
        for t in range((nc + te - 1) // te):
            if kind == "restrict":   # fine nodes of the tile's coarse elements and one below
                first, count, P, need = r * (t * te - 1), r * (te + 1), nf, r * nc
            else:                    # coarse nodes of the tile's coarse elements and the next
                first, count, P, need = te * t, te + 1, nc, nc + 1
            calls += [(i, P, int(i < need)) for i in range(first, first + count)]
    calls = sorted(set(calls))
    code = '#include "index_wrap.hpp"\n#include <cstdio>\nint main(){int c[][3]={' + \
        ",".join("{%d,%d,%d}" % c for c in calls) + \
        '};for(auto&v:c){int k=fep3m::wrap_tile(v[0],v[1]);' \
        'if(k<0||k>=v[1]||(v[2]&&k!=((v[0]%v[1])+v[1])%v[1]))std::printf("%d/%d/%d ",v[0],v[1],k);}}'
    assert _run(tmp_path, code) == []
    src = open(os.path.join(CSRC, "k_mesh.hip")).read()
    body = src[src.index("__global__ __launch_bounds__(256) void k_" + kind):]
    body = body[:body.index("__syncthreads")]
    assert "wrapi(" not in body and body.count("wrap_tile(") == 3   # the columns' three indices go through it


def test_march_tiles_stay_on_the_mesh(tmp_path):
    """Orders 3 to 6, 3 to 512 elements, 1 to 1024 configurations (2^28 elements in all), both kinds of plan: the
    plan's blocks cover the mesh, and the last input column of the last tile lies below 2 P, where one wrap gives
    an index of the axis."""
    code = r"""
#include "index_wrap.hpp"
#include "march_plan.hpp"
#include <cstdio>
using namespace fep3m;
int main() {
  for (int p = 3; p <= 6; ++p)
    for (int n = 3; n <= 512; ++n)
      for (int nb = 1; nb <= 1024 && std::int64_t(nb) * n * n * n <= (1 << 28); nb = nb < 8 ? nb + 1 : nb < 1024 ? nb + nb / 8 + 1 > 1024 ? 1024 : nb + nb / 8 + 1 : 1025)
        for (int shared = 0; shared < 2; ++shared)
          for (int sys = nb; sys <= 2 * nb; sys += nb) {
            const MarchPlan q = march_plan(p, n, nb, sys, shared);
            bool ok = q.nx * q.tx >= n && q.ny * q.ty >= n && q.nz * q.ze >= n && q.blocks() == q.nx * q.ny * q.nz;
            const int P = p * n, t[2] = {q.tx * q.nx, q.ty * q.ny};
            for (int k = 0; k < 2; ++k)   // columns -p .. t p of the axis
              for (int i = -p; i <= t[k] * p; ++i) {
                const int w = wrapi(i, P);
                ok = ok && w >= 0 && w < P;
              }
            if (!ok) std::printf("p%d_n%d_nb%d_%dx%d ", p, n, nb, q.tx, q.ty);
          }
}
"""
    assert _run(tmp_path, code) == []
