// Exact reflection symmetry of the near-field tables (host and device).
#pragma once

#include <cstddef>

#include "host_device.hpp"

namespace fep3m {

// The tables T[a][D][m] are symmetric under the axis reflections (offset, node
// and the sign of odd powers) but for the rounding of their solves.  Called for
// every entry i, in any order: the first of the up to eight entries that the
// reflections map onto each other replaces them all by their average.  Pairs
// are summed axis by axis, so that entries which must vanish do.
FEP3M_HOST_DEVICE inline void symmetrise_entry(size_t i, int p, int nl, int n_sr, double *T) {
  const int q1 = p + 1, S = 2 * n_sr + 1, M = q1 * q1 * q1, ND = S * S * S;
  const int m = int(i % M), D = int(i / M % ND), a = int(i / M / ND);
  const int mc[3] = {m % q1, m / q1 % q1, m / q1 / q1}, Dc[3] = {D % S, D / S % S, D / S / S};
  const int odd = (a % nl & 1) | (a / nl % nl & 1) << 1 | (a / nl / nl & 1) << 2;
  size_t at[8];
  double v[8], sg[8];
  for (int r = 0; r < 8; ++r) {
    int mr = 0, Dr = 0;
    for (int c = 2; c >= 0; --c) {
      mr = mr * q1 + (r >> c & 1 ? q1 - 1 - mc[c] : mc[c]);
      Dr = Dr * S + (r >> c & 1 ? S - 1 - Dc[c] : Dc[c]);
    }
    at[r] = (size_t(a) * ND + Dr) * M + mr;
    if (at[r] < i) return;
    const int b = r & odd;
    sg[r] = (b ^ b >> 1 ^ b >> 2) & 1 ? -1.0 : 1.0;
  }
  for (int r = 0; r < 8; ++r) v[r] = sg[r] * T[at[r]];
  const double t = 0.125 * (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
  for (int r = 0; r < 8; ++r) T[at[r]] = sg[r] * t;
}

}  // namespace fep3m
