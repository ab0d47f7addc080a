// The widths of the kernels' array offsets: 32-bit byte offsets where every offset that a kernel
// forms stays below 4 GB, else 64-bit ones (kWideMode). Host code without HIP, so that the bounds
// can be checked against the offsets themselves on any machine.
#pragma once

#include <algorithm>
#include <cstddef>

#include "lattice.hpp"

namespace lbm {

// Planes from the lower plane of a pair of opposite directions to the end of the upper one: the
// pulls, and the adjoint's scatter, address both planes of a pair from the lower one's base.
constexpr int pair_planes() {
  int reach = 0;
  for (int i = 0; i < D3Q19::Q; ++i) reach = std::max(reach, D3Q19::opp[i] - i);
  return reach + 1;
}

// Upper bounds of the byte offsets formed on a lattice of N nodes with planes `ps` elements apart (at
// least the fluid nodes), `s` bytes per stored population and `r` per value of the arithmetic type.
// Forward kernels: a stored population of a pair's upper plane, the 4-vectors per fluid id, the pairs of
// reals per node, and the launch lists (8 bytes per node).
constexpr size_t step_offsets(size_t N, size_t ps, size_t s, size_t r) {
  return std::max(std::max(pair_planes() * s * ps, 4 * r * ps), std::max(2 * r * N, 8 * N));
}
// Reverse kernels: the same, and an adjoint population of a pair's upper plane, which has the arithmetic
// type in every storage.
constexpr size_t adjoint_offsets(size_t N, size_t ps, size_t s, size_t r) {
  return std::max(step_offsets(N, ps, s, r), pair_planes() * r * ps);
}
constexpr bool wide(size_t offsets) { return offsets >= (size_t(1) << 32); }

}  // namespace lbm
