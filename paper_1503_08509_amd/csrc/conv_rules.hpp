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

// Complex values of the spectrum (one octant, na moments, M nodes) and of the
// work arrays of nb configurations.
inline size_t conv_spec_values(int N, int na, int M) {
  const size_t H = N / 2 + 1;
  return H * H * H * na * M;
}
inline size_t conv_work_values(int N, int na, int M, int nb) {
  return size_t(N) * N * N * nb * 2 * ((na + 1) / 2 + (M + 1) / 2);
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

}  // namespace fep3m
