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


def test_class_listing_covers_every_atom_once(lib):
    for scap in (1, 1024, 1025, 65536, 65537, 1024000):
        blocks = min(64, (scap + 1023) // 1024)
        for n in sorted({0, 1, min(scap, 1023), min(scap, 1024), scap // 3, scap - 1, scap}):
            span = lib.o3_order_span(n, blocks)
            assert span % 1024 == 0 and span * blocks >= n
            assert n == 0 or (span - 1024) * blocks < n  # no workgroup takes more than it must


def test_classes_only_for_several_species_and_contractions_that_pay_for_them(lib):
    for flops in (0.0, 1e5, 4e5, 6e5, 5e6):
        assert not lib.o3_classes(1, 16, flops)
        assert lib.o3_classes(2, 16, flops) == (flops >= 5e5)
        assert lib.o3_classes(2, 20, flops) == (flops >= 3e5)


@pytest.mark.parametrize("most", [1, 2, 4, 8, 16])
def test_splits_of_a_tile(lib, most):
    for grid in (16, 48, 256, 512):
        for ntile in (0, 1, 3, 15, 16, 31, 100, 255, 256, 257, 500, 512, 513, 9000):
            for fill in (0, 1):
                g = 1 << lib.o3_split_log(ntile, grid, most, fill)
                assert 1 <= g <= max(most, 1)
                if fill:  # the smallest that fills the grid
                    assert g == 1 or ntile * g // 2 < grid
                    assert g == most or ntile * g >= grid
                else:     # the largest that takes one round of it
                    assert g == 1 or ntile * g <= grid
                    assert g == most or 2 * ntile * g > grid


# Operations per S atom of the contraction: 8 and 12 radial functions at lmax 3 and
# 4, 16 at lmax 5 and 6 (sparse stage, dense stage)
LIGHT, USUAL, WIDE, WIDEST = (3.0e4, 6.0e4), (2.3e5, 4.9e5), (9.1e5, 2.15e6), (2.1e6, 3.9e6)


def test_cheap_potential_starts_late_only_beside_a_contraction_that_hides_it(lib):
    def late(form, reduced, ops, n, rebuild, classes=0):
        return bool(lib.fork_after_basis(form, lib.o3_weight(form, reduced, classes, *ops), n, rebuild))

    for n in (250, 2000, 8191, 54000, 1000000):
        assert not lib.fork_after_basis(0, 0.0, n, 0)  # no order-3 contraction
        assert not late(1, 0, LIGHT, n, 0)
        for form in (1, 3):
            assert late(form, 0, USUAL, n, 0) and late(form, 0, WIDE, n, 0)
        # the reverse slots of a call that rebuilds the list go on that stream too
        assert late(1, 0, USUAL, n, 1) == (n >= 100000)  # a long contraction covers both
        assert not late(1, 0, LIGHT, n, 1) and not late(3, 0, USUAL, max(n, 4000), 1)
        assert late(1, 0, WIDEST, n, 1)
        # two atom classes: not where the second's long tiles meet the cheap potential
        for ops in (USUAL, WIDEST):
            assert late(2, 0, ops, n, 0) and late(2, 0, ops, n, 0, classes=1)
            assert late(2, 0, ops, n, 1, classes=1) == (n <= 3000)
    # a contraction in between: a rebuilding call of few atoms
    assert [late(3, 0, USUAL, n, 1) for n in (2000, 4000)] == [True, False]
    assert [late(1, 0, WIDE, n, 1) for n in (2000, 4000)] == [True, False]


def test_fork_rule_is_monotonic_in_the_weight(lib):
    weights = [0.0] + [10 ** (4 + k / 16) for k in range(64)]
    for n in (1, 2048, 2049, 3000, 3001, 99999, 100000, 2000000):
        for form in (1, 2, 3):
            for rebuild in (0, 1):
                got = [lib.fork_after_basis(form, w, n, rebuild) for w in weights]
                assert got == sorted(got)
