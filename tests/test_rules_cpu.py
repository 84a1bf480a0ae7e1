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
    # a workgroup that counts the atoms before its own reads at most 15 others' share
    for scap in (1, 1024, 16384, 16385, 65536, 1024000):
        blocks = (scap + 1023) // 1024
        assert lib.o3_count_first(scap) == (blocks > 16)
        # the lists and the counts fit the pair gradients, three floats a slot
        assert scap + blocks <= 3 * scap
