"""Registers of the compiled kernels, read from the metadata that the compiler
left in the built library: a SIMD has 512 registers per lane, handed out in
eights, so the count sets how many wavefronts of a kernel it holds."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2502_19081_amd", "libmlmix.so")


def _notes(elf):
    """Metadata maps of an AMDGPU code object."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + k * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + k * size + 24)
        if kind != 7:  # SHT_NOTE
            continue
        p, end = off, off + length
        while p + 12 <= end:
            name_len, desc_len, note = struct.unpack_from("<III", elf, p)
            p += 12 + (name_len + 3 & ~3)
            if note == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[p:p + desc_len], strict_map_key=False)
            p += desc_len + 3 & ~3


@pytest.fixture(scope="module")
def kernels():
    """Mangled name -> (registers of a lane, bytes of scratch memory)."""
    if not os.path.exists(LIB):
        from paper_2502_19081_amd import build
        build.build()
    blob = open(LIB, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        p = m.end()
        count, = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" not in target or not size:
                continue
            for meta in _notes(blob[m.start() + off:m.start() + off + size]):
                for k in meta["amdhsa.kernels"]:
                    out[k[".name"]] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
    assert out
    return out


def _waves(kernels, pattern):
    got = {k: 512 // (v[0] + 7 & ~7) for k, v in kernels.items() if re.search(pattern, k)}
    assert got, pattern
    return got


# Every lmax and radial count of the vector pair adjoints: two wavefronts per
# SIMD in FP64, four in FP32 (their pairs' serial chains hide behind one another).
@pytest.mark.parametrize("name,at_least", [("k_ace_pairgrad_d", 2), ("k_ace_pairgrad_h", 4)])
def test_vector_pair_adjoints(kernels, name, at_least):
    got = _waves(kernels, name)
    assert len(got) == 7 * 4 * 2  # lmax, padded radial counts, single or batched
    assert min(got.values()) >= at_least, got
    assert all(kernels[k][1] == 0 for k in got)


# The workgroup pair adjoint at one channel tile: four, as many as its LDS
# leaves room for.
def test_workgroup_pair_adjoint(kernels):
    got = _waves(kernels, r"k_ace_pairgrad_wgILi1E")
    assert len(got) == 6 * 2  # lmax 0 .. 5, single or batched
    assert min(got.values()) >= 4, got
    assert all(kernels[k][1] == 0 for k in got)
