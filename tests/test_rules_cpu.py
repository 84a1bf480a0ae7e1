"""Dispatch rules over their whole range, on the CPU."""
import pytest

from tests import rules


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return rules.load(str(tmp_path_factory.mktemp("rules")))


def test_padded_radial_counts_and_their_lds(lib):
    for n_rad in range(1, 17):
        nr = lib.padded_nrad(n_rad)
        assert nr in (4, 8, 12, 16) and n_rad <= nr < n_rad + 4
        for ns in range(1, 9):
            nchp = (ns * n_rad + 3) // 4 * 4
            for lmax in range(7):
                l2 = (lmax + 1) ** 2
                if l2 * nchp > 1024:
                    continue  # refused when the model is made
                rows = l2 * ns * nr  # entries of an atom's padded row
                assert rows // nr < 512
                cap = 256
                assert 4 * (rows + cap // 2) * 8 <= 65536       # FP64: four rows and lists
                assert 4 * (2 * rows + 2 * cap) * 4 <= 65536    # FP32: eight rows and lists
                inv = (65536 + ns - 1) // ns
                assert all((r * inv) >> 16 == r // ns for r in range(l2 * ns))


def test_class_lists_count_before_they_rank_in_large_capacities(lib):
    # a workgroup that counts the atoms before its own reads at most 63 others' share
    for scap in (1, 1024, 16384, 65536, 65537, 1024000):
        blocks = (scap + 1023) // 1024
        assert lib.o3_count_first(scap) == (blocks > 64)
        # the lists and the counts fit the pair gradients, three floats a slot
        assert scap + blocks <= 3 * scap


def test_classes_only_for_several_species_and_contractions_that_pay_for_them(lib):
    for flops in (0.0, 1e5, 4e5, 6e5, 5e6):
        assert not lib.o3_classes(1, 16, flops)
        assert lib.o3_classes(2, 16, flops) == (flops >= 5e5)
        assert lib.o3_classes(2, 20, flops) == (flops >= 3e5)


@pytest.mark.parametrize("most", [1, 2, 4, 8, 16])
def test_splits_of_a_tile(lib, most):
    for grid in (16, 48, 256, 512):
        for ntile in (0, 1, 3, 15, 16, 31, 100, 255, 256, 257, 500, 512, 513, 9000):
            for fill in (1, 4, most):
                g = 1 << lib.o3_split_log(ntile, grid, most, fill)
                assert 1 <= g <= max(most, 1)
                if g > fill:  # one round of workgroups
                    assert ntile * g <= grid
                if g < most:  # no further split would still help
                    assert ntile * g * 2 > grid and (g >= fill or ntile * g >= grid)
