// Dispatch rules on sizes and types that need no device code: plain C++, so that
// they can be checked over their whole range without a GPU.
#pragma once

namespace mlmix {
namespace rules {

// Radial functions that the vector pair adjoints are compiled for: the model's
// count (1 .. 16) rounded up to a multiple of four, as the channels are.
constexpr int padded_nrad(int nrad) { return (nrad + 3) & ~3; }

// S atoms of a workgroup of the class listing: whole thousands (of 1024), equal for
// all of blocks workgroups.
constexpr int o3_order_span(int nS, int blocks)
{
    return ((nS + 1023) / 1024 + blocks - 1) / blocks * 1024;
}

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
// max_split of them: the largest split whose items run in one round of workgroups,
// or with fill the smallest that fills the grid.
constexpr int o3_split_log(int ntile, int grid, int max_split, bool fill)
{
    int lg = 0;
    while ((1 << lg) < max_split && (fill ? (long long)ntile << lg < grid : (long long)ntile << (lg + 1) <= grid))
        ++lg;
    return lg;
}

// Weight of an order-3 contraction for the fork rule below, in FP32 operations per S
// atom: form 1 the single-species form (its vector-ALU sparse stage runs at a third
// of the dense stage's rate, reduced operands at eight times it), 2 the wide form
// (slower per operation), 3 the FP64 form. In two classes the wide form weighs as
// much as lets a kept list start the cheap potential late and a rebuilding call of
// more than 3,000 atoms early: there the reverse slots delay the cheap potential
// until it meets the few long tiles of the second class, which need compute units
// to themselves (2 x 12 functions, lmax 4, 0.2 % of the second species, BF16, early /
// late: a rebuilding call on 54,000 atoms with a cylinder 720 / 872 us, on 11,664 with
// one defect 168 / 157; a kept list there 139 / 129).
constexpr double o3_weight(int form, bool reduced, bool classes, double sparse, double dense)
{
    return form == 2 ? (classes ? 3e6 : 4.0 * (sparse + dense))
                     : (form == 3 ? 3.0 : 1.0) * (3.0 * sparse + (reduced ? 0.125 : 1.0) * dense);
}

// Whether a mixed step of a single system starts the cheap potential on the second
// stream after the atomic basis, to run beside the order-3 contraction, instead of
// after the neighbour rows. Its workgroups (one wave per atom, all at once) keep the
// few blocks of the compaction and the basis waiting when they start first, and a
// long contraction hides them; after a short one they hold up the step's end.
// Measured early / late with both in one process (n_rad functions, lmax):
//  - a weight of 7e5 and more: FP32 12, 4 (1.2e6), 10 steps: 857 / 794 us on 2,000
//    atoms, 1,085 / 1,033 on 11,664, one defect; 16, 5 (4.9e6), a kept-list call: 105 / 102
//    us on 2,662, 402 / 375 on 128,000; FP64 12, 4 (3.5e6): 105 / 98 on 2,662; BF16 12, 4
//    (7.5e5), 10 steps: 805 / 784 on 2,662, 1,029 / 1,017 on 11,664;
//  - 4e5: FP32 12, 3, kept list: 139 / 144 us on 39,366, 335 / 323 on 128,000;
//  - below: FP32 8, 3 (1.5e5): 136 / 143 us on 39,366, 310 / 323 on 128,000;
//  - a call that rebuilds the list builds the reverse slots on that stream too, which
//    few contractions hide: FP32 12, 4: 82 / 93 us on 4,394, 113 / 120 on 11,664, but 78 /
//    77 on 2,000; FP64 12, 4 (3.5e6): 114 / 106 on 2,662, 153 / 161 on 11,664; FP32 16, 6
//    (1e7): 179 / 168 on 2,662, 317 / 298 on 39,366;
//  - a rebuilding call of 100,000 atoms and more, one vacancy per 6,000 atoms: FP32 16, 4
//    (1.6e6): 1,063 / 1,007 us on 128,000, 2,047 / 1,877 on 250,000, 9,013 / 8,414 on
//    1,024,000; BF16 16, 5 (3e6): 1,870 / 1,790 on 250,000 (with one defect 1,356 / 1,380); at
//    12, 3 (4e5) no difference. The FP64 form (2,341 / 2,464 on 250,000) and two atom
//    classes (BF16 2 x 12, 4: 2,475 / 2,890) stay early.
constexpr bool fork_after_basis(int form, double weight, int n, bool rebuild)
{
    if (rebuild)
        return weight >= 6.5e6 || (form == 1 && weight >= 7e5 && n >= 100000) || (weight >= 3e6 && n <= 3000) || (weight >= 1.3e6 && n <= 2048);
    return weight >= 7e5 || (weight >= 4e5 && n >= 100000);
}

}  // namespace rules
}  // namespace mlmix
