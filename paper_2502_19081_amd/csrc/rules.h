// Dispatch rules on sizes and types that need no device code: plain C++, so that
// they can be checked over their whole range without a GPU.
#pragma once

namespace mlmix {
namespace rules {

// Radial functions that the vector pair adjoints are compiled for: the model's
// count (1 .. 16) rounded up to a multiple of four, as the channels are.
constexpr int padded_nrad(int nrad) { return (nrad + 3) & ~3; }

// Class lists of the wide contraction: count the workgroups' atoms in a launch of
// its own (1.7 us of a step) above this S capacity. Below, a workgroup counts the
// atoms before it by itself, up to 64 rounds of them when S fills the capacity
// (about 20 us of the 1.2 ms and more that such a call takes), a few when it holds
// a tenth.
constexpr bool o3_count_first(int scap) { return scap > 65536; }

// Two atom classes in the wide contraction, for models of several species whose
// contraction takes at least this many operations per S atom: the listing and the
// second launch cost 6-8 us of an all-expensive call, the first class saves at most
// half of the contraction (more where it leaves out a channel tile). One class /
// two, all-expensive FP32 call on 2,000 atoms, host crystal of species 0 and alloy:
// 2 x 7 channels, lmax 3 (4.1e5): 87 / 86 and 97 / 104 us; 2 x 12, lmax 1 (1.5e5): 87 /
// 94 and 99 / 107; 2 x 16, lmax 1 (3.4e5): 116 / 111 and 136 / 143; 2 x 13, lmax 2
// (9.3e5): 125 / 102 and 161 / 168; 2 x 12, lmax 4 (4.8e6), 8,192 atoms: 1,181 / 477 and
// 1,689 / 1,702.
constexpr bool o3_classes(int n_species, int channels, double flops)
{
    return n_species > 1 && flops >= (channels > 16 ? 3e5 : 5e5);
}

// log2 of the workgroups that share a tile of the wide contraction, at most
// max_split of them: up to fill_split the smallest number that fills the grid,
// beyond it only one whose items still run in one round of workgroups.
constexpr int o3_split_log(int ntile, int grid, int max_split, int fill_split)
{
    int lg = 0;
    while ((1 << lg) < max_split && (((1 << lg) < fill_split && (long long)ntile << lg < grid) ||
                                     (long long)ntile << (lg + 1) <= grid))
        ++lg;
    return lg;
}

}  // namespace rules
}  // namespace mlmix
