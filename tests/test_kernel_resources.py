"""What the compiler made of kernels whose speed hangs on their registers, from the metadata of the library's own code objects.
No GPU needed."""
import struct

import msgpack
import pytest

from paper_2211_10280_amd import binding as B


def _sections(elf):
    """(name, type, bytes) of a 64-bit ELF file's sections"""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count, names = struct.unpack_from("<HHH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQ", elf, shoff + i * size) for i in range(count)]
    strings = elf[heads[names][4]:heads[names][4] + heads[names][5]]
    for name, kind, _, _, offset, length in heads:
        yield strings[name:strings.index(b"\0", name)].decode(), kind, elf[offset:offset + length]


def _kernels(elf):
    """the metadata of a code object's kernels: its AMDGPU note (type 32) is a map in MessagePack"""
    for _, kind, data in _sections(elf):
        at = 0
        while kind == 7 and at + 12 <= len(data):
            n, d, t = struct.unpack_from("<III", data, at)
            body = at + 12 + (n + 3) // 4 * 4
            if t == 32 and data[at + 12:at + 12 + n] == b"AMDGPU\0":
                yield from msgpack.unpackb(data[body:body + d])["amdhsa.kernels"]
            at = body + (d + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(B.LIB_PATH, "rb") as f:
        fat = b"".join(data for name, _, data in _sections(f.read()) if name == ".hip_fatbin")
    found, at = {}, 0
    while (at := fat.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        count, = struct.unpack_from("<Q", fat, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", fat, entry)
            if b"gfx950" in fat[entry + 24:entry + 24 + n]:
                found.update((k[".name"], k) for k in _kernels(fat[at + offset:at + offset + size]))
            entry += 24 + n
        at += 24
    return found


def test_narrow_updates_that_chain_long_rows_keep_their_registers(kernels):
    """Held to 6 waves per SIMD these kernels kept up to 24 registers of a lane in memory and took up to 7 % longer than the update
    with the chaining in a launch before it."""
    chaining = {n: k for n, k in kernels.items() if "k_apply_sub" in n and "ChainRider" in n}
    assert len(chaining) == 18                     # two types, three widths, three grids
    assert {n: k[".vgpr_spill_count"] for n, k in chaining.items() if k[".vgpr_spill_count"]} == {}


def test_keys_that_run_beside_a_forward_pass_are_small(kernels):
    """The keys of a large announced mini-batch find room among the waves of the forward pass before it: with 89 scalar registers
    instead of 62 (the list of centers alone in the same kernel) they took until its end, and calls up to 12 % longer."""
    keys = [k for n, k in kernels.items() if "k_prep_keys" in n]
    assert keys and all(k[".sgpr_count"] <= 72 and k[".vgpr_count"] <= 32 for k in keys)
