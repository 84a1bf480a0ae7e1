// Dispatch rules on sizes and types that need no device code: plain C++, so that
// they can be checked over their whole range without a GPU.
#pragma once

namespace mlmix {
namespace rules {

// Radial functions that the vector pair adjoints are compiled for: the model's
// count (1 .. 16) rounded up to a multiple of four, as the channels are.
constexpr int padded_nrad(int nrad) { return (nrad + 3) & ~3; }

}  // namespace rules
}  // namespace mlmix
