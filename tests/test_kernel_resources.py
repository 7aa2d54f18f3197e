"""Registers and scratch memory of the built kernels, read from the metadata of
libppl.so's own code objects (no GPU needed)."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2010_08454_amd", "libppl.so")


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in a shared library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + tlen]:
                yield blob[at + off:at + off + size]
            p += 24 + tlen
        at += len(magic)


def _kernels(elf):
    """The kernel records of an ELF code object's metadata note."""
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        _, kind, _, _, off, _ = struct.unpack_from("<IIQQQQ", elf, sections + k * size)
        if kind == 7:                                  # SHT_NOTE
            nlen, dlen, _ = struct.unpack_from("<III", elf, off)
            at = off + 12 + (nlen + 3) // 4 * 4
            yield from msgpack.unpackb(elf[at:at + dlen])["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels():
    with open(LIB, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}
    assert found, "no gfx950 kernels in the library"
    return found


def test_state_space_filter_keeps_its_state_in_registers(kernels):
    """Particles, log-weights and the noise drawn ahead stay in registers across
    the grid exchanges at every count of particles per lane."""
    mine = {n: k for n, k in kernels.items() if "smc_persistent_kernelINS_5LgssmE" in n}
    assert len(mine) == 8
    assert {n: k[".private_segment_fixed_size"] for n, k in mine.items()} == {n: 0 for n in mine}


def test_chains_keep_their_tables_in_registers(kernels):
    """Neither scratch memory nor an LDS table inside a Metropolis-Hastings
    iteration: the static LDS is the reduction's alone (30 sums of four waves, 8
    of four lanes for every row of 16)."""
    lds = {"mcmc_poly_kernelE": 30 * 4 * 8, "mcmc_poly_quad_kernelE": 16 * 4 * 8 * 8}
    for part, size in lds.items():
        k, = [k for n, k in kernels.items() if part in n]
        assert k[".private_segment_fixed_size"] == 0
        assert k[".group_segment_fixed_size"] == size


def test_enumeration_sums_do_not_depend_on_the_device(kernels):
    """The walk's workgroups, which group its FP64 sums, are a number of the
    library's own for every state and step count (asked here without a device),
    and it is the number that 256 CUs hold by the kernel's registers and LDS, at most
    2048 and one per tile of 128 prefixes."""
    import ctypes
    records = ctypes.CDLL(LIB)._ZN3ppl12enum_recordsEii
    for k in range(2, 9):
        for t in (t for t in range(1, min(40, 1024 // (k * k)) + 1) if k ** t <= 2 ** 50):
            nested = min({2: 12, 3: 7, 4: 6, 5: 5, 6: 5}.get(k, 4), t - 1)
            part = f"enum_sum_kernelILi{k}ELi{nested}E"
            kern, = [v for n, v in kernels.items() if part in n]
            waves = 512 // (-(-kern[".vgpr_count"] // 8) * 8)              # per SIMD, 512 registers in eights
            held = min(4 * waves // 2, 160 * 1024 // kern[".group_segment_fixed_size"])
            tiles = -(-k ** (t - nested) // 128)
            assert records(k, t) == min(tiles, 2048, 256 * held), (k, t)
