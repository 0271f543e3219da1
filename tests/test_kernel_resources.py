"""What the compiler gave the kernels of the built library, read from the metadata notes of its
code objects: no wave-tile kernel keeps registers in scratch memory, and the scalar ones that do not fit
(kept in lanes of vector registers, a vector instruction for each move) stay few."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

_BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 ELF images inside the library's offload bundles."""
    at = lib.find(_BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", lib, at + len(_BUNDLE))
        pos = at + len(_BUNDLE) + 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", lib, pos)
            name = lib[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name and size:
                yield lib[at + offset:at + offset + size]
        at = lib.find(_BUNDLE, pos)


def _kernels(elf):
    """The kernel entries of an image's NT_AMDGPU_METADATA note (type 32)."""
    assert elf[:4] == b"\x7fELF"
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        if kind != 7:                                                   # SHT_NOTE
            continue
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 0x18)
        pos, end = offset, offset + size
        while pos < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (namesz + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            pos = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    from paper_2506_15976_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2506_15976_amd import build
        build.build(force=True, verbose=False)
    with open(binding.LIB_PATH, "rb") as f:
        lib = f.read()
    return {k[".name"]: k for elf in _code_objects(lib) for k in _kernels(elf)}


def test_kernels_of_every_family_are_there(kernels):
    for family in ("wave_fwd_kernel", "wave_bwd_kernel", "chunk_fwd_kernel", "carry_chain_kernel", "reorder_kernel",
                   "reduce_partials_kernel", "conv1d_fwd_kernel", "conv1d_bwd_kernel"):
        assert any(family in name for name in kernels), family


def test_no_kernel_uses_scratch_memory(kernels):
    # (the chunk kernel's fp32 instances are held to three blocks a CU and spill 5 to 22 registers)
    spilling = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in kernels.items()
                if (k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]) and "chunk_fwd_kernelIf" not in n}
    assert not spilling


def test_forward_kernels_spill_few_scalars(kernels):
    # at most half the lanes of one vector register (with the ways of loading of all rows in one
    # kernel up to 68 were spilled, and a tile took a dozen vector instructions for them)
    spilling = {n: k[".sgpr_spill_count"] for n, k in kernels.items()
                if "wave_fwd_kernel" in n and k[".sgpr_spill_count"] > 32}
    assert not spilling
