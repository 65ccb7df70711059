// Periodic wrap of mesh indices (host and device).
#pragma once

namespace fep3m {

// Periodic wrap of an index known to lie in [-P, 2P).
constexpr int wrapi(int i, int P) { return i < 0 ? i + P : (i >= P ? i - P : i); }

// The same for a tile that may be wider than the mesh (its columns from 2P on
// feed only nodes that are not owned): some index of the axis there.
constexpr int wrap_tile(int i, int P) {
  const int k = wrapi(i, P);
  return k < P ? k : P - 1;
}

}  // namespace fep3m
