// Tiles and march lengths of the mesh operator of orders 3 to 6 (k_march.hip).
#pragma once

#include <cmath>
#include <cstdint>

namespace fep3m {

// A block's tile and march length.
struct MarchPlan {
  int tx, ty, ze;
  int nx, ny, nz;   // blocks per system along each axis
  constexpr int blocks() const { return nx * ny * nz; }
};

// The march length of least cost: rounds of resident blocks times the steps of
// one (the start of a march costs 0.6 of a step: one element's planes and
// carried rows), for sys systems.  resident: what the chip's 256 compute units
// hold, two blocks of the large tiles or four of the small.
inline MarchPlan plan_for(int n, int sys, int tx, int ty, int resident) {
  MarchPlan best{};
  double cost = 1e300;
  for (int ze = 1; ze <= 16 && ze <= n; ++ze) {
    MarchPlan q{tx, ty, ze, (n + tx - 1) / tx, (n + ty - 1) / ty, (n + ze - 1) / ze};
    const double r = double(sys) * q.blocks() / resident, rounds = std::ceil(r);
    const double c = (rounds < 4 ? rounds : r + 0.5) * (ze + 0.6);
    if (c < cost - 1e-9) {
      cost = c;
      best = q;
    }
  }
  return best;
}

// Whether a tile of t elements on a mesh of n reads columns below 2 P only, as
// wrapi needs: its last column is the first past its elements.  Every tile of
// 4 and fewer does (n >= 3); 8 on n = 3 and 4 does not.
constexpr bool tile_wraps(int n, int t) { return (n + t - 1) / t * t < 2 * n; }

// Tiles by order: large tiles re-read the fewest inputs, but a mesh that
// gives them fewer than 1.5 blocks per compute unit runs small ones, which
// spread over more of them (p = 5 on 8^3 elements: 5.1 us per launch
// against 6.9; on 16^3 13.1 against 11.7).  Order 3: 4 x 4 columns 14.2
// against 14.7 us for 8 x 4 on 32^3, 135 against 104 us on 64^3 (a Chebyshev
// step), where their rows of 12 nodes leave half of each cache line to others.
// In between neither is better throughout (whole evaluations with forces, 4 x 4
// and 8 x 4: 6.25 and 6.16 ms on 33^3, 8.75 and 8.94 on 40^3, 12.75 and 12.78 on
// 45^3, 14.72 and 14.72 on 48^3, 21.17 and 21.64 on 54^3, 32.99 and 32.24 on 64^3,
// by how the tiles divide the edge); the line is halfway.
//
// The length of the march suits the systems of the launch, except where sums
// over a block follow from it (the dot products and the fused restriction,
// shared): there a context of nb configurations keeps one plan, for 2 nb
// systems, so that the forward and adjoint systems give the same bits solved
// together or alone.  That plan leaves half of the chip idle for one system:
// 30 us per launch at p = 5, 27^3, and 26 with its own length.  (A shared
// length for both counts: 35 to 32 us for one system there, but 64 to 69 for
// two on 32^3.)
inline MarchPlan march_plan(int p, int n, int nb, int sys, bool shared) {
  const int64_t big = int64_t(2) * nb * ((n + 3) / 4) * ((n + 3) / 4) * n;   // blocks of 4 x 4 columns, one element each
  if (shared) sys = 2 * nb;
  switch (p) {
    case 3:
      return int64_t(2) * nb * n * n * n >= 131072 && tile_wraps(n, 8) ? plan_for(n, sys, 8, 4, 512)
                                                                       : plan_for(n, sys, 4, 4, 1024);
    case 4: return plan_for(n, sys, 4, 4, 512);
    case 5: return big >= 384 ? plan_for(n, sys, 4, 4, 512) : plan_for(n, sys, 2, 2, 1024);
    default: return plan_for(n, sys, 2, 2, 512);
  }
}

inline MarchPlan shared_plan(int p, int n, int nb) { return march_plan(p, n, nb, nb, true); }

}  // namespace fep3m
