// When near_field = AUTO takes the transforms of k_conv.hip, and on which lattice.
#pragma once

#include <cstddef>
#include <cstdint>

namespace fep3m {

constexpr int kConvMaxN = 72;

// N = r1 r2, each a radix that the passes have (up to 11 and 13): the split
// nearest to square, the larger factor first.
inline bool radices(int N, int &r1, int &r2) {
  r1 = r2 = 0;
  for (int d = 1; d <= 13; ++d) {
    if (d == 12 || N % d) continue;
    const int e = N / d;
    if (e > 13 || e == 12) continue;
    r1 = d;
    r2 = e;
    if (d >= e) return true;
  }
  return r1 > 0;
}

// Lattice edge for n elements (a box: padded by n_sr or more), or 0: none.
inline int conv_edge(int n, int nsr, bool box) {
  int r1, r2;
  if (n > 64) return 0;
  int N = box ? n + nsr : n;
  if (!box) return radices(N, r1, r2) ? N : 0;
  while (!radices(N, r1, r2)) ++N;   // at most 72 for n = 64
  return N;
}

// Complex values of the spectrum (one octant, na moments, M nodes).
inline size_t conv_spec_values(int N, int na, int M) {
  const size_t H = N / 2 + 1;
  return H * H * H * na * M;
}

// Whether the transforms' arrays may take `bytes` of device memory, `spectrum`
// of them the tables' spectrum: 32 GiB for the latter (the largest family on
// 64^3 elements, the 27-element q = 4 screens, takes 25 GB and gains the most,
// 399 to 127 ms per call with 10^6 charges), and in all a quarter of what is
// free at create.  Three quarters then stay for what the program allocates
// later, the graph's staging buffers and further contexts among it; work
// arrays, which grow with the batch, are bounded with the rest.  Beyond, the
// table sums, which need none.
constexpr size_t kConvSpecMax = size_t(32) << 30;
constexpr bool conv_memory(size_t spectrum, size_t bytes, size_t free_bytes) {
  return spectrum <= kConvSpecMax && bytes <= free_bytes / 4;
}

// Whether the transforms are the faster path, for nl moments per axis at order
// p.  With n_sr = 3 they are for every mesh, family and batch (at least 1.3
// times; 343 offsets per element against a few radix steps).  With n_sr = 1
// the table sums have 27 offsets, and on a chip that a large lattice or batch
// fills they win: near field and moment adjoint of the transforms and the sums,
// in ms, on 65536 elements as 16 configurations of 16^3: 27-element q = 1 0.29
// and 0.16, one-element q = 4 2.72 and 1.87, 27-element q = 4 14.3 and 7.0, a
// box (one-element q = 3) 1.06 and 0.52; on one 16^3 mesh 0.088 and 0.109, 0.29
// and 1.07, 1.14 and 3.86, 0.16 and 0.34.  The line is drawn in elements, per
// family at its crossing (8000 to 14000; 20000 to 33000; 64000 and 110000 to
// 125000): an element counts by the lattice it is padded to, squared, since the products'
// octants and the passes both grow with it, and from 27 moments on, where the
// sums are bound by arithmetic, by the share of their bricks of 4 x 4 x 8
// elements that the mesh fills (27-element q = 3, 1000 configurations of 5^3: 5.3
// and 13.6 ms).  With n_sr = 2 the sums win only in large batches of boxes whose
// bricks are full and whose lattice holds twice the elements (8^3 on 10^3, one-
// element q = 3, 256 configurations: 3.7 and 2.9 ms; 16 of them 0.29 and 0.98).
constexpr bool conv_pays(int n, int N, int nsr, int p, int nl, bool box, int nb) {
  const double el = double(n) * n * n, lattice = double(N) * N * N, pad = lattice / el;
  if (nsr == 1) {
    const int u = (n + 3) / 4 * 4, v = (n + 7) / 8 * 8;
    const double bricks = nl >= 3 ? double(u) * u * v / el : 1.0;
    const double line = nl == 1 ? 115000.0 : p == 3 ? 8192.0 : p == 4 || (p == 5 && nl > 2) ? 64000.0 : 20000.0;
    return nb * lattice * pad <= line * bricks;
  }
  return !(nsr == 2 && box && nl == 2 && n % 8 == 0 && pad > 1.9 && nb * lattice > 1e5);
}

}  // namespace fep3m
