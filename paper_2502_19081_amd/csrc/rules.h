// Dispatch rules on sizes and types that need no device code: plain C++, so that
// they can be checked over their whole range without a GPU.
#pragma once

namespace mlmix {
namespace rules {

// Radial functions that the vector pair adjoints are compiled for: the model's
// count (1 .. 16) rounded up to a multiple of four, as the channels are.
constexpr int padded_nrad(int nrad) { return (nrad + 3) & ~3; }

// Class lists of the wide contraction: count the workgroups' atoms in a launch of
// its own above this S capacity. Below, each of at most 16 workgroups counts at
// most 15 rounds of atoms itself, which costs what the launch would.
constexpr bool o3_count_first(int scap) { return scap > 16384; }

}  // namespace rules
}  // namespace mlmix
