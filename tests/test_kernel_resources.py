"""What the compiler says of the built kernels (the metadata notes of the library's own code object): registers that it had to
spill in kernels of the main path, where a run-time value in place of a constant has cost a tenth of the kernel before."""
import struct

import msgpack
import pytest

from paper_2509_16434_amd import learner as L


def _kernels():
    """{mangled name: its metadata} of the gfx950 code object in the library's offload bundle."""
    with open(L.LIB_PATH, "rb") as f:
        lib = f.read()
    at = lib.index(b"__CLANG_OFFLOAD_BUNDLE__")
    entries, p = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
    for _ in range(entries):
        off, size, n = struct.unpack_from("<QQQ", lib, p)
        target = lib[p + 24:p + 24 + n]
        p += 24 + n
        if target.endswith(b"gfx950"):
            elf = lib[at + off:at + off + size]
            headers, count = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<H", elf, 56)[0]
            for k in range(count):
                kind, _, note = struct.unpack_from("<IIQ", elf, headers + 56 * k)
                if kind == 4:   # PT_NOTE: name size, description size, type, name, description
                    nn, nd, ty = struct.unpack_from("<III", elf, note)
                    if ty == 32:   # NT_AMDGPU_METADATA
                        start = note + 12 + (nn + 3 & ~3)
                        return {m[".name"]: m for m in msgpack.unpackb(elf[start:start + nd])["amdhsa.kernels"]}
    raise AssertionError("no gfx950 metadata in " + L.LIB_PATH)


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def _of(kernels, prefix):
    found = {n: m for n, m in kernels.items() if n.startswith(prefix)}
    assert found, prefix
    return found


def test_row_length_of_the_known_width_stays_a_constant(kernels):
    """The register-fused input gradient of 80-wide rows: 27 spilled scalars, 174 where the loaders' row length is read at run time."""
    for n, m in _of(kernels, "_Z24k_conv_dgrad_wgrad0_tileILi1ELi8ELi80EE").items():
        assert m[".sgpr_spill_count"] <= 40 and m[".private_segment_fixed_size"] == 0, n


def test_forward_kernels_use_no_scratch(kernels):
    """64 channels to more than 64 in tiles of columns has the fewest registers left: the places of its results, kept apart from
    tile to tile, cost four of them spilled."""
    for n, m in _of(kernels, "_Z15k_conv_fwd_tile").items():
        assert m[".vgpr_spill_count"] == 0 and m[".private_segment_fixed_size"] == 0, n
